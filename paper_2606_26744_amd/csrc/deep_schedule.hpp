// Where the pinned K loop of gemm_deep.hip fetches from: plain integer rules, shared with a host
// test that walks the loop's loads.
#pragma once

namespace hdf {

constexpr int kDeepRing = 4;     // weight units in the register ring, kDeepRing - 1 issued ahead

// A unit is 32 of K: two 16-K blocks of 4096 bytes in a 128-row weight group, 64 bytes of an
// activation row; a pair of units is 64 of K.  The loop issues loads kDeepRing - 1 units and up
// to three pairs past the end of its K range, whose values nothing uses.  They re-read the last
// unit or pair: a scalar offset beyond the descriptor's end is not a defined way to keep a raw
// buffer load from memory (the range check need not cover it), so no offset ever leaves it.
constexpr int deep_last(int i, int n) { return i < n ? i : n - 1; }

// Scalar byte offset of the 16-K block ss of the unit that load slot u of nu fetches; a lane adds
// up to 4080 bytes and reads 16.  Units count from ku0, the split's first.
constexpr int deep_weight_offset(int ku0, int u, int nu, int ss) {
  return (ku0 + deep_last(u, nu)) * 8192 + ss * 4096;
}
// Bytes of a weight group up to the 64-K step k1, the split's end: its descriptor's size.
constexpr int deep_weight_bytes(int k1) { return k1 * 2 * 8192; }

// Scalar byte offset, in an activation row, of the pair that load slot pr of np fetches (128
// bytes).
constexpr int deep_act_offset(int ku0, int pr, int np) { return (ku0 / 2 + deep_last(pr, np)) * 128; }

}  // namespace hdf
