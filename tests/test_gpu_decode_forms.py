"""The small-batch tiles in every form, at the edges of their heights.

A launch's form (workgroups per CU, hence slots of the LDS ring) follows from
the tiles it expects, and from what the other phase runs.  Rows are added in
one order whatever the form, so all give the same bits: each form of the
staged bf16 tiles is compared with the register-direct ones, each form of the
FP8 tiles with four per CU, on experts of rows at the edges of the 32-row
blocks and of one to three tiles.  tests/test_decode_form.py checks, without a
GPU, that these shapes take the forms that they name; the tiles' values are
checked against the oracle elsewhere (four per CU and, at some shapes, the
other forms)."""

import numpy as np
import pytest

from synth import BF16, FP8

pytestmark = pytest.mark.gpu

ROWS = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 193, 0, 2, 40]
E, E0, E_LOC, T = 64, 8, len(ROWS), sum(ROWS)
E_FOUR = 1024  # a pool of which the same tokens are expected to touch few experts: four per CU

# (type, H, I, form of GEMM1, form of GEMM2).  K of GEMM1 is H, of GEMM2 I: bf16
# K % 2048 == 0 rotates the blocks' order, FP8 K % 512 == 0 gathers scales by four blocks.
SHAPES = [
    (BF16, 64, 2560, 8, 4), (BF16, 64, 5120, 6, 4), (BF16, 2048, 2560, 8, 4), (BF16, 2048, 5120, 6, 4),
    (BF16, 2560, 2048, 4, 8), (BF16, 5120, 2048, 4, 6), (BF16, 5120, 64, 4, 8), (BF16, 10240, 64, 4, 6),
    (BF16, 2048, 2048, 4, 4), (BF16, 192, 320, 4, 4),
    (FP8, 512, 2560, 8, 4), (FP8, 512, 5120, 6, 4), (FP8, 128, 2560, 8, 4), (FP8, 128, 5120, 6, 4),
    (FP8, 5120, 512, 4, 8), (FP8, 10240, 512, 4, 6), (FP8, 5120, 384, 4, 8), (FP8, 10240, 128, 4, 6),
    (FP8, 384, 640, 4, 4),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class _Layer:
    """A context over device-made inputs whose resident experts get exactly ROWS
    tokens each, in both phases (k = 1: out is y, by token)."""

    def __init__(self, dtype, H, I, experts=E, t_p=T, d_priority_us=0):
        import torch

        from paper_2609_00993_amd import moepd as M

        gen = torch.Generator(device="cuda")
        gen.manual_seed(56)
        w, scales = [], [None, None]
        for i, (n, K) in enumerate(((2 * I, H), (H, I))):
            v = torch.randn((E_LOC, n, K), generator=gen, device="cuda")
            if dtype == FP8:
                w.append((v * 16).to(torch.float8_e4m3fn).view(torch.uint8))
                scales[i] = torch.randint(115, 120, (E_LOC, n, K // 32), generator=gen, dtype=torch.uint8, device="cuda")
            else:
                w.append((v * K ** -0.5).to(torch.bfloat16))
        owner = E0 + np.random.default_rng(57).permutation(np.repeat(np.arange(E_LOC), ROWS))
        logits = torch.full((max(T, t_p), experts), -1.0, device="cuda")
        logits[torch.arange(T, device="cuda"), torch.from_numpy(owner).cuda()] = 1.0
        self.M, self.logits, self.keep = M, logits, (w, scales)
        self.x = torch.randn((max(T, t_p), H), generator=gen, device="cuda").to(torch.bfloat16)
        self.out = [torch.full((t, H), float("nan"), device="cuda") for t in (max(T, t_p), T)]
        torch.cuda.synchronize()
        cfg = M.make_config(experts, E0, E_LOC, 1, H, I, M.MOE_DTYPE_FP8 if dtype == FP8 else M.MOE_DTYPE_BF16,
                            max(T, t_p), T, d_priority_us=d_priority_us)
        st, self.ctx = M.moe_ctx_create(cfg, *w, *scales)
        M.check(st, "moe_ctx_create")
        self.streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def enqueue(self, ph, t=T, stream=None):
        self.M.layer(self.ctx, ph, self.logits, t, self.x, self.out[ph], stream or self.streams[ph])

    def run(self, ph, t=T):
        import torch

        self.out[ph].fill_(float("nan"))
        torch.cuda.synchronize()
        self.enqueue(ph, t)
        torch.cuda.synchronize()
        return self.out[ph][:t].clone()

    def close(self):
        self.M.check(self.M.moe_ctx_destroy(self.ctx))


@pytest.mark.parametrize("dtype,H,I,form1,form2", SHAPES)
def test_forms_give_the_same_bits(dtype, H, I, form1, form2):
    import torch

    prefill = 32 * E  # tokens of a P batch on large tiles: D's bf16 tiles are then register-direct
    g = _Layer(dtype, H, I, t_p=prefill)
    try:
        got = g.run(1)
        assert torch.isfinite(got).all() and bool(got.abs().max() > 0)
        if dtype == BF16:
            g.run(0, prefill)
            assert torch.equal(g.run(1), got)
    finally:
        g.close()
    if dtype == FP8:
        g = _Layer(dtype, H, I, experts=E_FOUR)
        try:
            assert torch.equal(g.run(1), got)
        finally:
            g.close()


@pytest.mark.parametrize("dtype,H,I", [(BF16, 192, 320), (BF16, 2048, 2048), (BF16, 2560, 768), (FP8, 512, 640),
                                       (FP8, 384, 512), (FP8, 2560, 768)])
def test_forms_beside_the_other_phase(dtype, H, I):
    """Both phases small under D-first admission: P takes the form that leaves
    D's tiles room once D has run, and a D layer captured after a small P batch
    the form that fits there.  Each gives the bits of a context that runs its
    phase alone, also while both run."""
    import torch

    g = _Layer(dtype, H, I)
    try:
        alone = [g.run(0), None]
    finally:
        g.close()
    g = _Layer(dtype, H, I, d_priority_us=500)
    try:
        alone[1] = g.run(1)
        assert torch.equal(g.run(0), alone[0])
        graph, sg = torch.cuda.CUDAGraph(), g.streams[1]
        with torch.cuda.graph(graph, stream=sg):
            g.enqueue(1, stream=sg)
        for rep in range(3):
            for o in g.out:
                o.fill_(float("nan"))
            torch.cuda.synchronize()
            g.enqueue(0)
            with torch.cuda.stream(sg):
                graph.replay()
            torch.cuda.synchronize()
            for ph in (0, 1):
                assert torch.equal(g.out[ph][:T], alone[ph]), (rep, ph)
        del graph
    finally:
        g.close()


def test_small_d_tiles_beside_256_row_tiles():
    """D's staged tiles while P runs 256-row tiles whose GEMM2 is the hand-over
    pair, at a width where two 32-column blocks make a D tile (K not a multiple
    of 2048): the bits of each phase alone."""
    import torch

    H, I, wide = 512, 768, 512 * E
    g = _Layer(BF16, H, I, t_p=wide)
    try:
        alone = [g.run(0, wide), g.run(1)]
    finally:
        g.close()
    g = _Layer(BF16, H, I, t_p=wide, d_priority_us=500)
    try:
        g.run(0, wide)
        g.run(1)
        for rep in range(3):
            for o in g.out:
                o.fill_(float("nan"))
            torch.cuda.synchronize()
            g.enqueue(0, wide)
            for _ in range(4):
                g.enqueue(1)
            torch.cuda.synchronize()
            for ph in (0, 1):
                assert torch.equal(g.out[ph], alone[ph]), (rep, ph)
    finally:
        g.close()
