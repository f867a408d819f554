"""Weights and scales at bases with no more than their element's alignment (a
view into a packed checkpoint): the GEMMs read them in 16-byte pieces, from
registers and by LDS DMA, which take any byte address.  Every tile regime
gives the bits it gives for aligned copies of the same values."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _place(t, offset):
    """A copy of t that starts `offset` bytes into an aligned buffer, and its address."""
    import torch

    raw = t.contiguous().view(torch.uint8).reshape(-1)
    buf = torch.zeros(raw.numel() + 256, dtype=torch.uint8, device="cuda")
    buf[offset:offset + raw.numel()] = raw
    return buf, buf.data_ptr() + offset


def _layer(dtype, H, I, T, phase, w_off, s_off):
    import torch

    from paper_2609_00993_amd import moepd as M

    E, k = 16, 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(55)
    keep, scales = [], [(None, None), (None, None)]
    x_type = torch.float32 if dtype == "f32" else torch.bfloat16
    for i, (n, K) in enumerate(((2 * I, H), (H, I))):
        w = torch.randn((E, n, K), generator=gen, device="cuda")
        if dtype == "fp8":
            keep.append(_place((w * 16).to(torch.float8_e4m3fn).view(torch.uint8), w_off))
            s = torch.randint(117, 120, (E, n, K // 32), generator=gen, dtype=torch.uint8, device="cuda")
            scales[i] = _place(s, s_off)
        else:
            keep.append(_place((w * K ** -0.5).to(x_type), w_off))
    x = torch.randn((T, H), generator=gen, device="cuda").to(x_type)
    logits = torch.randn((T, E), generator=gen, device="cuda")
    out = torch.zeros((T, H), device="cuda")
    types = {"f32": M.MOE_DTYPE_F32, "bf16": M.MOE_DTYPE_BF16, "fp8": M.MOE_DTYPE_FP8}
    torch.cuda.synchronize()
    cfg = M.make_config(E, 0, E, k, H, I, types[dtype], 4096, 64)
    st, ctx = M.moe_ctx_create(cfg, keep[0][1], keep[1][1], scales[0][1], scales[1][1])
    M.check(st, "moe_ctx_create")
    try:
        M.layer(ctx, phase, logits, T, x, out, torch.cuda.Stream())
        torch.cuda.synchronize()
    finally:
        M.check(M.moe_ctx_destroy(ctx))
    return out


# small, prefill and 256-row tiles; K a multiple of 512 (scales of four steps in one gather) or not
@pytest.mark.parametrize("T,phase", [(24, 1), (700, 0), (4096, 0)])
@pytest.mark.parametrize("H,I", [(512, 512), (384, 640)])
@pytest.mark.parametrize("dtype,w_off,s_off", [("f32", 4, 0), ("bf16", 2, 0), ("bf16", 8, 0), ("fp8", 1, 0),
                                               ("fp8", 0, 1), ("fp8", 4, 2), ("fp8", 0, 8)])
def test_bits_do_not_depend_on_the_weights_alignment(dtype, w_off, s_off, H, I, T, phase):
    import torch

    ref = _layer(dtype, H, I, T, phase, 0, 0)
    assert bool(ref.abs().max() > 0)
    assert torch.equal(_layer(dtype, H, I, T, phase, w_off, s_off), ref)
