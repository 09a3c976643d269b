// The matrix-core bound tiles (bf16, more than 128 rows): C = A . W^T over the packed weight
// layout described in gemm.hip, 4 waves of TM x TN blocks of 32 x 32, one wave per SIMD, each
// with all rows of the tile:
//   TM = 4, TN = 4: 128 rows x 512 columns, a wave owns one 128-row weight group;
//   TM = 8, TN = 2: 256 rows x 256 columns, a wave owns half a weight group;
//   TM = 4, TN = 2: 128 rows x 256 columns, half the area at 1.18 times its share of the time,
//     for problems that do not fill whole rounds of the large tiles.
//
// K loop.  A unit is 32 of K, two sub-steps of 16 (8) MFMAs, which keep the matrix core of a
// SIMD busy for 1024 (512) cycles; sixteen accumulators fill the accumulation registers.
//   Weights: 8 KB a unit and block of TN, straight into a register ring of R units, issued
//     R - 1 units before their use.
//   Activations: loaded two units (64 of K, whole 128-byte lines) at a time, stored into
//     swizzled LDS unit buffers CU units before their use; one workgroup barrier per CU units.
//     A wave reads the fragments of a sub-step during the sub-step before it.
// With one wave per SIMD nothing hides a wait, so every load, LDS access and MFMA is pinned
// in the order it is written here (a scheduling fence after each): the compiler's own order
// sank the fragment reads to their uses, an exposed LDS round trip every four MFMAs.
// Addresses cost no vector instructions: buffer loads with a per-lane offset computed once
// and the unit in the scalar offset.  The activations' descriptor ends at the last row, so rows
// past M (a lane offset past its end) read as zero without a fetch; units past K, which the ring
// issues and nothing uses, re-read the last one (deep_schedule.hpp).
//
// Measured alone (random operands, warm): 16384 x 4096 -> 8192 972 -> 815 us with fp32 stores,
// 16384 x 16384 -> 4096 1878 -> 1520 us, 1024 x 4096 -> 24576 in two K splits 204 -> 180 us,
// 1024 x 12288 -> 4096 in four 96 -> 81 us (before: compiler-ordered loop of the 128 x 512
// tiles).  With the other epilogues, same box: keys and values 838 us (846 at the least and 870
// on average inside the cold step), bf16 rows 830, argmax 779, fp32 rows 837.  Copies without
// stores run at 1.40-1.52 PFLOP/s, without any load from memory in the loop at 1.60-1.72, the
// MFMAs alone at 1.67-1.80 (the power limit on such data).
#include "common.hpp"
#include "deep_schedule.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace hdf {

constexpr int kDeepThreads = 256;
// Row tiles of one group in the tile order of tall problems: consecutive tile ids walk four
// row tiles of a column block, then the next column block, so that the 32 tiles an XCD runs
// share activation and weight slices in its L2 (16384 x 4096 -> 8192: 4 row tiles 846 us, 8
// 889, 2 887, 1 895; 16384 x 16384 -> 4096 within 1% from 1 to 4, 8 3% slower).  Up to eight
// row tiles form one group, so that weights from HBM are fetched by all of them at once (1024
// rows as eight tiles of 128: 24576 columns 193 us in one group, 207 in two).
constexpr int kDeepGroup = 4;

typedef __amdgpu_buffer_rsrc_t BufRsrc;
__device__ __forceinline__ BufRsrc buf_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 buf_ld16(BufRsrc r, int lane_off, int uniform_off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, uniform_off, 0));
}
// Nothing moves across (the pinned order of the K loop).
#define HDF_PIN() __builtin_amdgcn_sched_barrier(0)

// 16-byte chunk c (8 of K) of a unit's row r sits at chunk c ^ unit_swizzle(r), so that the
// stores (eight threads a row, four in each of two units) and the fragment reads (32 rows,
// one chunk each) meet distinct banks.
__device__ __forceinline__ int unit_swizzle(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }

template <int TM_, int TN_>
struct DeepTile {
  static constexpr int TM = TM_, TN = TN_;
  static constexpr int BM = 32 * TM, BN = 128 * TN;
  static constexpr int UK = 32;
  static constexpr int CU = TM == 4 ? 4 : 2;            // units per barrier
  static constexpr int NB = 2 * CU;                     // LDS unit buffers
  static constexpr int UB = BM * UK + 32;               // elements between them: 64 bytes apart in
                                                        // the banks, so that the two halves of a
                                                        // row's store do not meet (128 bytes: 25%
                                                        // of the LDS cycles were conflicts, now 0)
  static constexpr int PCH = BM * 64 * 2 / 16 / kDeepThreads;   // 16-byte chunks a thread and pair
  static constexpr size_t kLds = size_t(NB) * UB * sizeof(bf16_t);
};

// acc[i][t] += rows 32i.. of the tile x columns of the wave's block t, over units ku0 ..
// ku0 + nu - 1 (nu even, at least 2).  The first half of the blocks lies from byte off0 of
// every 16 K of rb0 on, the second from off1 of rb1.  SWAP: the transposed product (the weights
// as the A operand).  On return every wave has left the loop's last LDS read behind, not a
// barrier.
template <int TM, int TN, bool SWAP>
__device__ __forceinline__ void deep_loop(f32x16_t (&acc)[TM][TN], const BufRsrc ra_, int64_t lda,
                                          const BufRsrc rb0, int off0, const BufRsrc rb1, int off1,
                                          int ku0, int nu, bf16_t* lds) {
  using Tl = DeepTile<TM, TN>;
  constexpr int UK = Tl::UK, CU = Tl::CU, NB = Tl::NB, UB = Tl::UB, PCH = Tl::PCH;
  constexpr int R = kDeepRing, D = R - 1, AH = PCH / 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int bv0 = lane * 16 + off0, bv1 = lane * 16 + off1;
  int av[PCH], al[PCH];   // chunk q of a pair: row q/8, 16-byte column q%8 (unit q%8/4)
#pragma unroll
  for (int j = 0; j < PCH; ++j) {
    const int q = tid + kDeepThreads * j, row = q >> 3, c = q & 7;
    av[j] = row * int(lda) * 2 + c * 16;
    al[j] = (c >> 2) * UB + row * UK + (((c & 3) ^ unit_swizzle(row)) * 8);
  }
  // Fragment of sub-step ss, row block i: lane l reads row 32i + l%32, chunk 2ss + l/32.
  const int fr = lane & 31;
  int fo[2];
#pragma unroll
  for (int ss = 0; ss < 2; ++ss) fo[ss] = fr * UK + (((2 * ss + (lane >> 5)) ^ unit_swizzle(fr)) * 8);
  u32x4 rb[R][2][TN];
  u32x4 ra[2][PCH];
  const int np = nu / 2;
  auto a_load = [&](int pr, int j, u32x4* dst) {
    dst[j] = buf_ld16(ra_, av[j], deep_act_offset(ku0, pr, np));
  };
  auto b_load = [&](int u, int ss, int t, u32x4 (*dst)[TN]) {
    const int at = deep_weight_offset(ku0, u, nu, ss);
    dst[ss][t] = t < TN / 2 ? buf_ld16(rb0, bv0 + t * 1024, at) : buf_ld16(rb1, bv1 + (t - TN / 2) * 1024, at);
  };
  auto a_store = [&](const u32x4* src, int j, int buf) {
    *reinterpret_cast<u32x4*>(&lds[buf * UB + al[j]]) = src[j];
  };
  auto frag = [&](int buf, int ss, int i) {
    return *reinterpret_cast<const bf16x8_t*>(&lds[buf * UB + fo[ss] + 32 * i * UK]);
  };
  auto mma = [](bf16x8_t act, u32x4 w, f32x16_t c) {
    const bf16x8_t wv = __builtin_bit_cast(bf16x8_t, w);
    return SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, act, c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_32x32x16_bf16(act, wv, c, 0, 0, 0);
  };
  // Prologue: the pairs of the first CU units into LDS (they are waited for first), the next
  // pair and the first D units of weights in flight.
  u32x4 first[CU / 2][PCH];
#pragma unroll
  for (int v = 0; v < CU / 2; ++v)
#pragma unroll
    for (int j = 0; j < PCH; ++j) a_load(v, j, first[v]);
#pragma unroll
  for (int j = 0; j < PCH; ++j) a_load(CU / 2, j, ra[0]);
#pragma unroll
  for (int x = 0; x < D; ++x)
#pragma unroll
    for (int ss = 0; ss < 2; ++ss)
#pragma unroll
      for (int t = 0; t < TN; ++t) b_load(x, ss, t, rb[x]);
#pragma unroll
  for (int v = 0; v < CU / 2; ++v)
#pragma unroll
    for (int j = 0; j < PCH; ++j) a_store(first[v], j, 2 * v);
  lds_barrier();
  bf16x8_t f0[TM], f1[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) f0[i] = frag(0, 0, i);
  // Unit u, with j = u % U known at compile time.  During it: this unit's second fragments
  // and the next unit's first ones, half of the pair CU units ahead into LDS, half of the
  // loads of the pair after that one, the weights D units ahead; spread over the MFMAs.
  constexpr int U = 2 * CU > R ? 2 * CU : R;
  static_assert(U % R == 0 && U % NB == 0, "unit indexes are static over the unrolled units");
  auto unit = [&](int u, int j) {
    const int s = j % R, buf = j % NB, nbuf = (j + 1) % NB;
    const int wbuf = ((j / 2 + CU / 2) * 2) % NB;
    const int h = (j & 1) * AH, rs = (j / 2) & 1;
    auto rd1 = [&](int i) { f1[i] = frag(buf, 1, i); HDF_PIN(); };
    auto rd0 = [&](int i) { f0[i] = frag(nbuf, 0, i); HDF_PIN(); };
    auto st = [&](int x) { a_store(ra[rs], h + x, wbuf); HDF_PIN(); };
    auto la = [&](int x) { a_load((u >> 1) + CU / 2 + 1, h + x, ra[rs ^ 1]); HDF_PIN(); };
    auto lb = [&](int ss, int t) { b_load(u + D, ss, t, rb[(s + D) % R]); HDF_PIN(); };
    constexpr int NM = TM * TN;
#pragma unroll
    for (int k = 0; k < NM; ++k) {
      if constexpr (TM == 4 && TN == 4) {
        if (k < 8 && k % 2 == 0) rd1(k / 2);
        if (k < 12 && k % 3 == 1) lb(0, k / 3);
        if (k == 9 || k == 11) st((k - 9) / 2);
        if (k == 13 || k == 15) la((k - 13) / 2);
      } else if constexpr (TM == 4) {
        if (k < 4) rd1(k);
        if (k == 1 || k == 5) lb(0, k / 4);
        if (k == 4 || k == 6) st((k - 4) / 2);
        if (k == 5 || k == 7) la((k - 5) / 2);
      } else {
        if (k % 2 == 0) rd1(k / 2);
        if (k % 4 == 1) st(k / 4);
        if (k % 4 == 3) la(k / 4);
        if (k == 6 || k == 12) lb(0, (k - 6) / 6);
      }
      acc[k / TN][k % TN] = mma(f0[k / TN], rb[s][0][k % TN], acc[k / TN][k % TN]);
      HDF_PIN();
    }
    if (j % CU == CU - 1) {
      lds_barrier();
      HDF_PIN();
    }
#pragma unroll
    for (int k = 0; k < NM; ++k) {
      if constexpr (TM == 4 && TN == 4) {
        if (k < 8 && k % 2 == 0) rd0(k / 2);
        if (k % 4 == 3) lb(1, k / 4);
      } else if constexpr (TM == 4) {
        if (k < 4) rd0(k);
        if (k == 4 || k == 6) lb(1, (k - 4) / 2);
      } else {
        if (k % 2 == 0) rd0(k / 2);
        if (k == 5 || k == 11) lb(1, (k - 5) / 6);
      }
      acc[k / TN][k % TN] = mma(f1[k / TN], rb[s][1][k % TN], acc[k / TN][k % TN]);
      HDF_PIN();
    }
  };
  int u = 0;
  for (; u + U <= nu; u += U) {
#pragma unroll
    for (int j = 0; j < U; ++j) unit(u + j, j);
  }
#pragma unroll
  for (int j = 0; j < U; ++j)
    if (u + j < nu) unit(u + j, j);
}

// ---------------------------------------------------------------------------- epilogues
// Accumulator element r of block (i, t): product A.W^T: row 32i + 8(r/4) + 4(lane/32) + r%4,
// column 32t + lane%32 of the wave; transposed product: row 32i + lane%32, column
// 32t + 8(r/4) + 4(lane/32) + r%4.

// fp32 C (or split-K partial) straight from the accumulators.
template <int TM, int TN>
__device__ __forceinline__ void store_partial(const f32x16_t (&acc)[TM][TN], const GemmArgs& p, int z,
                                              int m0, int c0) {
  const int lane = threadIdx.x & 63;
  float* C = p.C + int64_t(z) * p.M * p.N;
#pragma unroll
  for (int t = 0; t < TN; ++t) {
    const int col = c0 + 32 * t + (lane & 31);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < p.M && col < p.N) C[int64_t(row) * p.N + col] = acc[i][t][r];
      }
  }
}

// Context K rows from the transposed product: a lane holds four consecutive dims of a row
// and, in another of its blocks, the four dims half a head on, so RoPE needs no exchange; four
// dims are 8 bytes of the key tile and the 64 lanes' runs are two pieces of 256 bytes.
// rows[]: cache row (-1: not stored) of the tile's rows; tab: the rotation table's rows of
// the tile, both in LDS.  16384 rows x 4096 in the cold step of 8 x 2048: 1010 -> 890 us for
// the launch (before: two waves a SIMD in ping-pong, 128 columns at a time through LDS).
constexpr int kRopeLd = 132;   // floats between the table rows in LDS

__device__ __forceinline__ void store_keys(const f32x16_t (&acc)[4][4], const GemmArgs& p, int c0,
                                           const int* rows, const float* tab) {
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const int HD = p.hd, HALF = HD >> 1;
  const bool wide = HD == 128;
  const bool rope = p.rope_cs != nullptr;
  // Block pair q: (0, 2), (1, 3) of one head of 128, or (0, 1), (2, 3) of two heads of 64.
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float* cs = tab + (32 * i + (lane & 31)) * kRopeLd + 8 * h;
    const int drow = rows[32 * i + (lane & 31)];
    const int rr = drow & 31;
    const int64_t base = int64_t(drow >> 6) * 64 * HD +
                         ((2 * ((drow & 63) >> 5) + ((rr >> 2) & 1)) * (HD >> 5) * 64 + 4 * (rr >> 3) + (rr & 3)) * 8 +
                         4 * h;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      bf16_t* kh = static_cast<bf16_t*>(p.kc) + int64_t(wide ? c0 / 128 : c0 / 64 + q) * p.cap * HD + base;
      const int slice = wide ? q : 0;   // 32-dim slice of the first half
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float y1[4], y2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x16_t& a = wide ? acc[i][q] : acc[i][2 * q];
          const f32x16_t& b = wide ? acc[i][2 + q] : acc[i][2 * q + 1];
          y1[e] = a[4 * g + e];
          y2[e] = b[4 * g + e];
        }
        if (rope) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float4 c = *reinterpret_cast<const float4*>(cs + ((wide ? 32 * q : 0) + 8 * g) * 2 + 4 * e);
            rope_rotate(y1[2 * e], y2[2 * e], c.x, c.y);
            rope_rotate(y1[2 * e + 1], y2[2 * e + 1], c.z, c.w);
          }
        }
        if (drow >= 0) {
          bf16_t* dst = kh + (slice * 64 + g * 16) * 8;
          *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf2(y1[0], y1[1]), pack_bf2(y1[2], y1[3]));
          *reinterpret_cast<uint2*>(dst + (HALF >> 5) * 512) =
              make_uint2(pack_bf2(y2[0], y2[1]), pack_bf2(y2[2], y2[3]));
        }
      }
    }
  }
}

// Context V rows, from the transposed product too (one K loop for the kernel): a lane holds
// four consecutive dims of a row; where a quad's four rows are four consecutive cache rows
// that start at a multiple of 4, the quad turns its 4 x 4 values round (two exchanges of
// packed pairs), so that each lane stores four rows of one dim, 8 bytes of the value tile;
// single elements otherwise.
__device__ __forceinline__ void store_values(const f32x16_t (&acc)[4][4], const GemmArgs& p, int c0,
                                             const int* rows) {
  const int lane = threadIdx.x & 63, h = lane >> 5, j = lane & 3;
  const int HD = p.hd;
  // Bytes of {partner, own} that give this lane (row j, row j^1) in row order of one dim of a pair.
  const uint32_t sel = (j & 1) ? 0x03020706u : 0x05040100u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int4 d = *reinterpret_cast<const int4*>(rows + 32 * i + (lane & 28));
    const bool run = d.x >= 0 && (d.x & 3) == 0 && d.y == d.x + 1 && d.z == d.x + 2 && d.w == d.x + 3;
    const int own = j == 0 ? d.x : j == 1 ? d.y : j == 2 ? d.z : d.w;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int col = c0 + 32 * t;
      bf16_t* vh = static_cast<bf16_t*>(p.vtc) + int64_t(col / HD) * p.cap * HD;
      const int dim0 = col % HD + 4 * h;
      const f32x16_t& a = acc[i][t];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t lo = pack_bf2(a[4 * g], a[4 * g + 1]), hi = pack_bf2(a[4 * g + 2], a[4 * g + 3]);
        // Even lanes then hold dims 0 and 2 of their and the next row, odd lanes 1 and 3 ...
        const uint32_t y0 = __builtin_amdgcn_perm(__builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true), lo, sel);
        const uint32_t y1 = __builtin_amdgcn_perm(__builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true), hi, sel);
        // ... and lane j dim j of all four rows.
        const uint32_t got = __builtin_amdgcn_mov_dpp(j < 2 ? y1 : y0, 0x4E, 0xF, 0xF, true);
        const uint2 four = j < 2 ? make_uint2(y0, got) : make_uint2(got, y1);
        const int dim = dim0 + 8 * g;
        if (run) {
          *reinterpret_cast<uint2*>(vh + vc_index(d.x, dim + j, HD)) = four;
        } else if (own >= 0) {
          vh[vc_index(own, dim, HD)] = bf16_t(lo);
          vh[vc_index(own, dim + 1, HD)] = bf16_t(lo >> 16);
          vh[vc_index(own, dim + 2, HD)] = bf16_t(hi);
          vh[vc_index(own, dim + 3, HD)] = bf16_t(hi >> 16);
        }
      }
    }
  }
}

// Row maxima (lowest column on ties) of the transposed product: over a lane's registers,
// across the lane halves by a shuffle, across the waves in LDS, one atomic per row into the
// row's packed key.  The logits leave, when asked for, block by block through a region of LDS
// of the wave's own.  129280 columns of 4096: 1024 rows 940 -> 826 us, 512 rows 493 -> 443, 300
// rows 377 -> 338, 2048 rows 1837 -> 1613 (before: ping-pong tiles of 128 x 512).
template <int TM, int TN>
__device__ __forceinline__ void fold_argmax(const f32x16_t (&acc)[TM][TN], const GemmArgs& p, int m0,
                                            int c0, float* lds) {
  constexpr int BM = 32 * TM;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, h = lane >> 5, tok = lane & 31;
  float best[TM];
  int bcol[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    best[i] = -INFINITY;
    bcol[i] = 0x7FFFFFFF;
  }
#pragma unroll
  for (int t = 0; t < TN; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int col = c0 + 32 * t + 8 * (r >> 2) + 4 * h + (r & 3);
      const bool in = col < p.N;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const float v = acc[i][t][r];
        const bool take = in & (v > best[i]);
        best[i] = take ? v : best[i];
        bcol[i] = take ? col : bcol[i];
      }
    }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const float ov = __shfl_xor(best[i], 32, kWave);
    const int oc = __shfl_xor(bcol[i], 32, kWave);
    if (ov > best[i] || (ov == best[i] && oc < bcol[i])) {
      best[i] = ov;
      bcol[i] = oc;
    }
  }
  lds_barrier();   // the K loop's last reads
  float* rv = lds;                                        // [wave][row] maxima
  int* rc = reinterpret_cast<int*>(lds + 4 * BM);         // [wave][row] columns
  if (lane < 32) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      rv[wid * BM + 32 * i + tok] = best[i];
      rc[wid * BM + 32 * i + tok] = bcol[i];
    }
  }
  lds_barrier();
  for (int row = threadIdx.x; row < BM; row += kDeepThreads) {
    float bv = rv[row];
    int bc = rc[row];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float ov = rv[w * BM + row];
      const int oc = rc[w * BM + row];
      if (ov > bv || (ov == bv && oc < bc)) {
        bv = ov;
        bc = oc;
      }
    }
    if (m0 + row < p.M && bc != 0x7FFFFFFF) atomicMax(p.keys + m0 + row, argmax_key(bv, bc));
  }
  if (p.C == nullptr) return;
  constexpr int LDC = 33;
  float* own = lds + 8 * BM + wid * 32 * LDC;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int t = 0; t < TN; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) own[tok * LDC + 8 * (r >> 2) + 4 * h + (r & 3)] = acc[i][t][r];
      __builtin_amdgcn_wave_barrier();
      const int col = c0 + 32 * t + tok;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + 32 * i + 2 * r + h;
        const float v = own[(2 * r + h) * LDC + tok];
        if (row < p.M && col < p.N) p.C[int64_t(row) * p.N + col] = v;
      }
      __builtin_amdgcn_wave_barrier();
    }
}

// bf16 rows (+ bias per column, fp32) from the transposed product, 32 rows at a time through
// a region of LDS of the wave's own, so that whole lines of a row leave together (stores
// straight from the registers meet half lines: 16384 x 4096 -> 8192 883 us that way against
// 837 for fp32 rows, 835 this way).
template <int TM, int TN>
__device__ __forceinline__ void store_rows(const f32x16_t (&acc)[TM][TN], const GemmArgs& p, int m0,
                                           int c0, bf16_t* lds) {
  constexpr int W = 32 * TN, LD = W + 8;        // columns of a wave, padded LDS row
  constexpr int PER = W / 8, RPI = 64 / PER;    // 16-byte pieces of a row, rows a store
  const int lane = threadIdx.x & 63, h = lane >> 5, tok = lane & 31;
  bf16_t* own = lds + (threadIdx.x >> 6) * 32 * LD;
  float* bias = reinterpret_cast<float*>(lds + 4 * 32 * LD);   // of the tile's columns
  lds_barrier();   // the K loop's last reads
  for (int c = threadIdx.x; c < 4 * W; c += kDeepThreads) {
    const int col = c0 - (threadIdx.x >> 6) * W + c;
    bias[c] = p.bias != nullptr && col < p.N ? p.bias[col] : -0.f;   // x + -0 is x
  }
  lds_barrier();
  bias += (threadIdx.x >> 6) * W + 4 * h;
  bf16_t* out = static_cast<bf16_t*>(p.out);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16_t& a = acc[i][t];
        const float4 b = *reinterpret_cast<const float4*>(bias + 32 * t + 8 * g);
        *reinterpret_cast<uint2*>(own + tok * LD + 32 * t + 8 * g + 4 * h) =
            make_uint2(pack_bf2(a[4 * g] + b.x, a[4 * g + 1] + b.y),
                       pack_bf2(a[4 * g + 2] + b.z, a[4 * g + 3] + b.w));
        HDF_PIN();
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 32 / RPI; ++q) {
      const int r = q * RPI + lane / PER, c = (lane % PER) * 8;
      const u32x4 v = *reinterpret_cast<const u32x4*>(own + r * LD + c);
      const int row = m0 + 32 * i + r, col = c0 + c;
      if (row < p.M && col < p.N) st16(out + int64_t(row) * p.N + col, v);   // N is a multiple of 8
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// The gated activation SiLU(gate) * up in bf16 from the transposed product: the first half of a
// wave's blocks are gate columns and the second half the same columns' up part, so that both
// meet in a lane.  Rows leave through a region of LDS of the wave's own, as in store_rows.
template <int TM, int TN>
__device__ __forceinline__ void store_gated(const f32x16_t (&acc)[TM][TN], const GemmArgs& p, int m0,
                                            int c0, bf16_t* lds) {
  constexpr int W = 16 * TN, LD = W + 8;        // columns of a wave, padded LDS row
  constexpr int PER = W / 8, RPI = 64 / PER;    // 16-byte pieces of a row, rows a store
  const int lane = threadIdx.x & 63, h = lane >> 5, tok = lane & 31;
  bf16_t* own = lds + (threadIdx.x >> 6) * 32 * LD;
  bf16_t* out = static_cast<bf16_t*>(p.out);
  const int F = p.N / 2;
  lds_barrier();   // the K loop's last reads
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int t = 0; t < TN / 2; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x16_t &a = acc[i][t], &b = acc[i][t + TN / 2];
        *reinterpret_cast<uint2*>(own + tok * LD + 32 * t + 8 * g + 4 * h) =
            make_uint2(pack_bf2(silu_mul(a[4 * g], b[4 * g]), silu_mul(a[4 * g + 1], b[4 * g + 1])),
                       pack_bf2(silu_mul(a[4 * g + 2], b[4 * g + 2]), silu_mul(a[4 * g + 3], b[4 * g + 3])));
        HDF_PIN();
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 32 / RPI; ++q) {
      const int r = q * RPI + lane / PER, c = (lane % PER) * 8;
      const u32x4 v = *reinterpret_cast<const u32x4*>(own + r * LD + c);
      const int row = m0 + 32 * i + r, col = c0 + c;
      if (row < p.M && col < F) st16(out + int64_t(row) * F + col, v);   // F is a multiple of 64
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <int TM, int TN, int EPI>
__global__ void __launch_bounds__(kDeepThreads, 1)
gemm_deep_kernel(GemmArgs p) {
  using Tl = DeepTile<TM, TN>;
  constexpr int BM = Tl::BM, BN = Tl::BN;
  static_assert(EPI != kEpiKV || (TM == 4 && TN == 4), "whole heads a wave");
  __shared__ __attribute__((aligned(16))) unsigned char smem[Tl::kLds];
  __shared__ __attribute__((aligned(16))) int row_tab[EPI == kEpiKV ? BM : 4];
  __shared__ __attribute__((aligned(16))) float rope_tab[EPI == kEpiKV ? BM * kRopeLd : 4];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // Tiles of the first problem, then those of the optional second one.
  const int tiles1 = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
  int tile = remap_tile(blockIdx.x, gridDim.x);
  if (tile >= tiles1) {
    tile -= tiles1;
    p.A = p.A2;
    p.lda = p.lda2;
    p.B = p.B2;
    p.M = p.M2;
    p.N = p.N2;
    p.C = p.C2;
  }
  const int mt = (p.M + BM - 1) / BM, nt = (p.N + BN - 1) / BN;
  const int group = mt <= 2 * kDeepGroup ? mt : kDeepGroup;
  const int in_group = group * nt;
  const int g = tile / in_group, first = g * group;
  const int gm = min(mt - first, group);
  const int gr = tile - g * in_group;
  const int m_tile = first + gr % gm, n_tile = gr / gm;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int nk_all = p.K / 64;
  const int z = blockIdx.z;
  const int k0 = (nk_all * z) / gridDim.z, k1 = (nk_all * (z + 1)) / gridDim.z;
  // This wave's 32-row weight blocks start at block blk0 of the packed weights (a group past
  // the last one is clamped to it, and the columns it computes are never stored).
  const int blk0 = (n_tile * 4 + wid) * TN;
  const int grp = min(blk0 >> 2, ((p.N + 127) >> 7) - 1);
  const bf16_t* A = static_cast<const bf16_t*>(p.A) + int64_t(m0) * p.lda;
  const bf16_t* B = static_cast<const bf16_t*>(p.B) + int64_t(grp) * (p.K >> 4) * 2048;
  const BufRsrc ra = buf_rsrc(A, int((int64_t(min(BM, p.M - m0) - 1) * p.lda + p.K) * 2));
  const BufRsrc rb = buf_rsrc(B, deep_weight_bytes(k1));
  const int off = (blk0 & 3) * 1024;
  // kEpiGated: a tile is BN / 2 gate columns and the same up columns; the wave's gate blocks
  // start at block gb, its up blocks F/32 blocks on (F is a multiple of 64, so two blocks of
  // one kind are in one 128-row group).  Blocks past F are clamped and never stored.
  BufRsrc rb0 = rb, rb1 = rb;
  int off0 = off, off1 = off + TN / 2 * 1024;
  if constexpr (EPI == kEpiGated) {
    const int fb = p.N / 64;
    const int gb = min((n_tile * 4 + wid) * (TN / 2), fb - TN / 2), ub = gb + fb;
    const bf16_t* W = static_cast<const bf16_t*>(p.B);
    rb0 = buf_rsrc(W + int64_t(gb >> 2) * (p.K >> 4) * 2048, deep_weight_bytes(k1));
    rb1 = buf_rsrc(W + int64_t(ub >> 2) * (p.K >> 4) * 2048, deep_weight_bytes(k1));
    off0 = (gb & 3) * 1024;
    off1 = (ub & 3) * 1024;
  }
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.f;
  bf16_t* lds = reinterpret_cast<bf16_t*>(smem);
  const int c0 = n0 + 32 * TN * wid;   // the wave's first column
  if constexpr (EPI == kEpiKV) {
    // Cache rows of the tile's rows and, for K, their rotation table rows, copied whole rows
    // at a time (the epilogue's lanes reading them from memory would touch 32 rows a load)
    // before the K loop, whose first loads they precede (copied after it: 9 us a tile).  Visible
    // after the K loop's barriers.
    if (threadIdx.x < BM) {
      const int row = m0 + threadIdx.x;
      row_tab[threadIdx.x] = row < p.M ? p.plan_row[row] : -1;
    }
    if (n0 < p.kv_d && p.rope_cs != nullptr) {
      const int per = p.hd >> 2;   // 16-byte pieces of a table row
#pragma unroll 8
      for (int q = threadIdx.x; q < BM * per; q += kDeepThreads) {
        const int r = q / per, c = q - r * per;
        const int pos = max(p.plan_pos[min(m0 + r, p.M - 1)], 0);   // -1: a row that is not stored
        *reinterpret_cast<u32x4*>(rope_tab + r * kRopeLd + 4 * c) =
            ld16(p.rope_cs + int64_t(pos) * p.hd + 4 * c);
      }
    }
  }
  constexpr bool SWAP = EPI != kEpiPartial;
  if (k1 > k0)
    deep_loop<TM, TN, SWAP>(acc, ra, p.lda, rb0, off0, rb1, off1, k0 * 2, (k1 - k0) * 2, lds);
  if constexpr (EPI == kEpiKV) {
    // d is a multiple of the tile's 512 columns, so a tile lies wholly in K or in V.
    if (n0 < p.kv_d)
      store_keys(acc, p, c0, row_tab, rope_tab);
    else
      store_values(acc, p, c0 - p.kv_d, row_tab);
  } else if constexpr (EPI == kEpiArgmax) {
    fold_argmax<TM, TN>(acc, p, m0, c0, reinterpret_cast<float*>(smem));
  } else if constexpr (EPI == kEpiGated) {
    store_gated<TM, TN>(acc, p, m0, (n_tile * 4 + wid) * 16 * TN, reinterpret_cast<bf16_t*>(smem));
  } else if constexpr (EPI == kEpiRows) {
    store_rows<TM, TN>(acc, p, m0, c0, reinterpret_cast<bf16_t*>(smem));
  } else {
    store_partial<TM, TN>(acc, p, z, m0, c0);
  }
}

// ---------------------------------------------------------------------------- host side

template <int TM, int TN, int EPI>
static void launch_deep(const GemmArgs& a, int splits, hipStream_t s) {
  using Tl = DeepTile<TM, TN>;
  const int tiles = ((a.M + Tl::BM - 1) / Tl::BM) * ((a.N + Tl::BN - 1) / Tl::BN) +
                    ((a.M2 + Tl::BM - 1) / Tl::BM) * ((a.N2 + Tl::BN - 1) / Tl::BN);
  hipLaunchKernelGGL((gemm_deep_kernel<TM, TN, EPI>), dim3(tiles, 1, splits), dim3(kDeepThreads), 0, s, a);
}

template <int EPI>
static void launch_tile(const GemmArgs& a, const GemmPlan& plan, int splits, hipStream_t s) {
  if (plan.bm == 256)
    launch_deep<8, 2, EPI>(a, splits, s);
  else if (plan.tn == 4)
    launch_deep<4, 4, EPI>(a, splits, s);
  else
    launch_deep<4, 2, EPI>(a, splits, s);
}

hipError_t launch_gemm_deep(int epi, const GemmArgs& a, const GemmPlan& plan, hipStream_t s) {
  if (epi == kEpiKV)
    launch_deep<4, 4, kEpiKV>(a, 1, s);
  else if (epi == kEpiArgmax && plan.bm == 256)
    launch_deep<8, 2, kEpiArgmax>(a, 1, s);
  else if (epi == kEpiArgmax)
    launch_deep<4, 4, kEpiArgmax>(a, 1, s);
  else if (epi == kEpiRows)
    launch_tile<kEpiRows>(a, plan, 1, s);
  else if (epi == kEpiGated)
    launch_tile<kEpiGated>(a, plan, 1, s);
  else
    launch_tile<kEpiPartial>(a, plan, plan.splits, s);
  return hipGetLastError();
}

// Tile shape and K split by the least estimated time: rounds of workgroups over the CUs, each
// its units of K (0.72 us for the large tiles, 0.415 for 128 x 256) and 5 us of start and end,
// plus the fp32 partials of every split, written here and read by the next kernel (5.2 TB/s).
// 1024 rows, with that reader: 4096 -> 24576 206 us as 256 x 256 tiles in two splits, 196 as
// 128 x 256 in one; 12288 -> 4096 83 in four splits, 80 in two (and half the partials);
// 4096 -> 4096 38 and 32; 4096 -> 20480 171 as 256 x 256 in one, 142.  Of the large shapes, 256
// x 256 up to 2048 rows, where the weights come from HBM and half as many row tiles re-read
// them (1024 x 4096 -> 24576 in two splits: 180 against 212 us; -> 129280 862 against 938),
// 128 x 512 above, whose fragments cost half the LDS reads (16384 x 4096 -> 8192: 815 against
// 820 us, 16384 x 16384 -> 4096 1520 against 1553), unless the other one takes fewer rounds.
static GemmPlan deep_plan(int M, int N, int M2, int N2, int K, int max_splits, double part, double* time) {
  const int ncu = device_cu_count();
  const int nk = K / 64;
  const bool tall = M > 2048 || M2 > 2048;
  struct Shape { int bm, tn; double unit; };
  const Shape shapes[3] = {{tall ? 128 : 256, tall ? 4 : 2, 0.72}, {tall ? 256 : 128, tall ? 2 : 4, 0.73},
                           {128, 2, 0.415}};
  GemmPlan best{4, 1, 2};
  best.bm = 256;
  double best_t = 1e30;
  for (int sp = 1; sp <= max_splits && (sp == 1 || nk / sp >= 8) && part * sp < best_t; ++sp)
    for (const Shape& x : shapes) {
      const int bn = 128 * x.tn;
      const int64_t tiles = ((int64_t(M) + x.bm - 1) / x.bm) * ((N + bn - 1) / bn) +
                            ((int64_t(M2) + x.bm - 1) / x.bm) * ((N2 + bn - 1) / bn);
      const double rounds = double((tiles * sp + ncu - 1) / ncu);
      const double t = rounds * (2.0 * ((nk + sp - 1) / sp) * x.unit + 5.0) + part * sp;
      if (t < best_t) {
        best_t = t;
        best = GemmPlan{4, sp, x.tn};
        best.bm = x.bm;
      }
    }
  if (time != nullptr) *time = best_t;
  return best;
}

GemmPlan deep_plan(int M, int N, int M2, int N2, int K) {
  return deep_plan(M, N, M2, N2, K, 8, (double(M) * N + double(M2) * N2) * 8.0 / 5.2e6, nullptr);
}

// The gate and up product with its activation in the epilogue (one K split, no partials): taken
// where its estimate is below that of partial sums and the pass over them (about 4 us and the
// partials' reads, which deep_plan counts).  1024 rows of 4096, 12288 wide: 175 + 19 -> 179 us;
// a few hundred rows of a narrow drafter leave most CUs without a tile in one split.
bool deep_gated_plan(int M, int F, int K, GemmPlan* plan) {
  double one = 0.0, split = 0.0;
  *plan = deep_plan(M, 2 * F, 0, 0, K, 1, 0.0, &one);
  (void)deep_plan(M, 2 * F, 0, 0, K, 8, double(M) * 2 * F * 8.0 / 5.2e6, &split);
  return one < split + 4.0;
}

// The LM head's tile: 256 x 256, whose weights half as many row tiles re-read from HBM (8 to
// 9% faster at equal rows), unless 128-row tiles pad the rows by that much less.
GemmPlan deep_argmax_plan(int M) {
  const int64_t pad256 = (int64_t(M) + 255) / 256 * 256, pad128 = (int64_t(M) + 127) / 128 * 128;
  const bool low = pad128 * 109 < pad256 * 100;
  GemmPlan p{4, 1, low ? 4 : 2};
  p.bm = low ? 128 : 256;
  return p;
}

}  // namespace hdf
