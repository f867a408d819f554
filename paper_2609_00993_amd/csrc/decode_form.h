// Forms of the small-batch tiles of both GEMMs (bf16 and MX FP8): one wave per
// workgroup, a ring of K blocks in LDS, and how many workgroups run on a CU.
// Host arithmetic and constants only, so that a test without a GPU can check
// which form a launch takes and that the forms fit as they claim.
#pragma once

#include <math.h>

namespace moepd {

// A CU's LDS and the units it is handed out in: of workgroups of 27,296 bytes
// five ran on a CU at once, of 26,880 six.
constexpr int kLdsPerCu = 160 * 1024;
constexpr int kLdsUnit = 1280;
constexpr int lds_units(int bytes) { return (bytes + kLdsUnit - 1) / kLdsUnit; }

// Workgroups per CU of the staged forms (kDecodeRoom: four, see below);
// kDecodeDirect: operands straight into registers, no LDS (bf16 only).
enum DecodeForm : int { kDecodeDirect = 0, kDecodeRoom = 1, kDecodeFour = 4, kDecodeSix = 6, kDecodeEight = 8 };

// LDS bytes of a workgroup.  Eight: what one slot of the tallest tile takes (bf16 96
// rows, FP8 64 rows and their scales).
constexpr int decode_lds(int form, bool mx) {
  return form == kDecodeFour ? 40960
         : form == kDecodeSix ? (mx ? 26880 : 24576)
         : form == kDecodeEight ? (mx ? 18432 : 20480)
                                : 33280;
}

// Small batches of both phases under D-first admission.  P's tiles wait for a D
// layer on their CUs, so what they hold must leave D's kernels room, however many of
// them a CU takes: kDecodeRoom fits four times and leaves 30 KB, a tile of D's
// form of six.  Without that room D's tiles wait for P's and P's for D, until
// P's wait budget ends.  Layer pair / D's layer in us, 500 us budget, P + D tokens,
// synchronised after each pair: P six or eight per CU and D eight (FP8 D by its
// tiles) -> these forms:
//   bf16, H 7168, 32 experts    700 + 4  755 / 364 -> 748 / 288   64 + 64  967 / 649 -> 1053 / 670
//   bf16, H 2560, 64 experts    700 + 64 795 / 693 -> 348 / 169   64 + 64  646 / 544 ->  278 / 179
//   bf16, H 2048, 32 experts    200 + 64 229 / 124 -> 241 / 136   64 + 64  229 / 129 ->  235 / 133
//   FP8, H 7168, 32 experts     700 + 64 1167 / 1036 -> 697 / 386
//   FP8, H 2560, 64 experts     700 + 64 745 / 647 -> 257 / 122
// P takes this form, and waits, once the context has run a D layer, since a D layer
// may start at any time; D takes its form while P has work in flight.
enum class Beside { kNone, kLeaveRoom, kFit };

// m-tiles of a small batch under even routing: the experts it touches, one
// standard deviation above the mean (a few tiles more than one round holds cost a
// second one).
inline double decode_m_tiles(int experts, int local_experts, int top_k, int T) {
  const double miss = pow(1.0 - (double)top_k / experts, (double)T), loc = local_experts;
  return fmin(loc, loc * (1.0 - miss) + sqrt(loc * miss * (1.0 - miss)));
}

// The staged form of a launch that expects `tiles` tiles.  Four (three slots of a
// 32-row tile) while they hold all the expected tiles, so that few waves keep
// enough in flight (256 GEMM1 tiles 46 us, 89 with eight), or while their last round
// is nearly full (skewed 2048 GEMM1 tiles 391 us, 414 with eight; beside the other
// phase's tiles, where few waves fit, D's layer 847 / 909 us).  Else eight with one
// slot (the block being multiplied is in registers meanwhile) while these run at
// once (1470 GEMM1 tiles 225 us, 252 with four; 0.15 of a round passes unnoticed),
// or six if its last round is the fuller (2560 GEMM2 tiles 51 / 58 us).
inline DecodeForm decode_form(double tiles, Beside beside) {
  if (beside == Beside::kLeaveRoom) return kDecodeRoom;
  if (beside == Beside::kFit) return kDecodeSix;
  auto rounds = [&](int per_cu) { return tiles / (256.0 * per_cu); };
  auto cost = [&](int per_cu) { return ceil(rounds(per_cu) - 0.15) / rounds(per_cu); };
  if (tiles <= 4 * 256 || cost(4) <= 1.1) return kDecodeFour;
  if (rounds(8) > 1.15 && cost(6) < cost(8)) return kDecodeSix;
  return kDecodeEight;
}

}  // namespace moepd
