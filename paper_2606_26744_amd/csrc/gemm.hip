// Dense contractions of the drafter step: C[M][N] = A[M][K] . W[N][K]^T with fp32
// accumulation.  A (activations) is row-major; W (weights) is stored in the
// MFMA-packed layout of hdf_pack_weight:
//   element (n, k) at (((n/128)*(K/16) + k/16)*4 + (n%128)/32)*512
//                     + ((n%32) + 32*((k%16)/8))*8 + k%8
// i.e. every block of 32 rows x 16 k is 512 elements laid out in exactly the order
// the 64 lanes of a wave hold the B operand of v_mfma_f32_32x32x16_bf16 (lane l: row
// l%32, k 8*(l/32)..+7), and the four 32-row blocks of a 128-row group sit side by
// side for every 16 k.  A wave streams its weights straight from HBM into registers
// with one contiguous 1 KB load per instruction, the four waves of a workgroup read
// one contiguous 16 KB run per 64-k step, and no weight byte passes through LDS.
//
// bf16 kernel: NW waves (4, 6 or 8), each owning TN 32-column blocks (1; 2 for the LM
// head's weight stream of up to 128 rows) and all BM rows (BM = 128, or 64 when M <= 64;
// 192 for the LM head's one-pass tiles) of a 32*NW*TN-column tile.  The activation slice
// (BM x 64) is shared through a double-buffered, padded LDS tile.  A ring of STAGES
// K-steps of weights is in flight per wave; activations are fetched one step further
// ahead than weights because memory counters complete in issue order.  The matrix-core
// bound problems (more than 128 rows; the LM head above 192) run in gemm_deep.hip.
// Split-K runs over gridDim.z; tiles are ordered so that the M-tiles of one weight
// column block run on the same XCD back to back (its L2 serves the re-reads).
//
// Epilogues:
//   PARTIAL  fp32 C (or split-K partial z at C + z*M*N) straight from registers
//   ARGMAX   LM head: the transposed product, so that per row (max, lowest index) is
//            taken over a lane's registers, then across the two lane halves and the
//            waves in LDS, and folded into a packed 64-bit key with one atomicMax per
//            row and tile; the logits are stored only when asked for
//
// fp32: the same kernel's plain K loop on v_mfma_f32_32x32x2_f32 with 4 waves of one
// 32-column block and 32, 64 or 128 rows (notes at the code).
#include <initializer_list>

#include "common.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace hdf {

constexpr int kBK = 64;        // K granularity of the bf16 tiles (K % kBK == 0)
constexpr int kShortSteps = 32;   // K steps up to which the stream plan weighs steps against partials
constexpr int kBKf32 = 32;     // K step of the fp32 tiles (K % 16 == 0; a last half step is zero-filled)

// TN: 32-column weight blocks per wave, 1, or 2 in the LM head's stream.  Each activation
// fragment read from LDS feeds TN matrix-core operations, so wider waves cut the LDS traffic
// per MFMA; the split weight streams prefer more waves per CU instead.
// NT: fetch the weights with non-temporal loads (they stream past the caches).  Right
// when one row tile reads every weight byte once; with several row tiles the others
// re-read the weights from L2, so they are fetched through the caches.
// T = float: the same tiles, rings and epilogues on v_mfma_f32_32x32x2_f32.  A K step is 128
// bytes of every activation row in either type, so the fp32 step is 32 of K; a packed
// 32 x 16 block is 32 bytes a lane (two loads), and lane l's eight values (row l%32, k
// 8*(l/32)..+7) are the operands of eight MFMAs, each taking k pair (e, 8 + e).
template <typename T, int BM, int NW, int STAGES, int EPI, int TN, bool NT>
__global__ void __launch_bounds__(NW * 64)
gemm_kernel(GemmArgs p) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int THREADS = NW * 64;
  constexpr int TM = BM / 32;
  constexpr int NB = NW * TN;                     // 32-column blocks of a tile
  constexpr int BN = 32 * NB;
  constexpr int BK = F32 ? kBKf32 : kBK;
  constexpr int VEC = 16 / int(sizeof(T));        // elements of a 16-byte chunk
  constexpr int LDA = BK + VEC;                   // padded LDS row (elements)
  constexpr int A_CHUNKS = BM * BK / VEC;          // 16-byte chunks of an activation step
  constexpr int A_CH = (A_CHUNKS + THREADS - 1) / THREADS;
  constexpr int LDC = 33;                         // padded row of a wave's 32 columns
  static_assert(EPI == kEpiPartial || NB % 4 == 0, "argmax tiles are whole 128-column slabs");
  // LDS: the activation buffers, reused after the K loop by the ARGMAX epilogue to stage the
  // logits 128 columns at a time ([block][row][32 columns]) and for its per-wave row maxima.
  constexpr size_t kMainLds = size_t(2) * BM * LDA * sizeof(T);
  constexpr size_t kEpiLds = EPI != kEpiPartial ? size_t(4) * BM * LDC * sizeof(float) : 0;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kMainLds > kEpiLds ? kMainLds : kEpiLds];
  typedef T ATile[BM][LDA];
  ATile* As = reinterpret_cast<ATile*>(smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wid = tid >> 6;

  // Tiles of the first problem, then those of the optional second one.
  const int tiles1 = ((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
  int tile = remap_tile(blockIdx.x, gridDim.x);
  const bool second = tile >= tiles1;
  if (second) {
    tile -= tiles1;
    p.A = p.A2;
    p.lda = p.lda2;
    p.B = p.B2;
    p.M = p.M2;
    p.N = p.N2;
    p.C = p.C2;
  }
  const int mt = (p.M + BM - 1) / BM;
  const int n_tile = tile / mt, m_tile = tile % mt;
  const int m0 = m_tile * BM, n0 = n_tile * BN;

  const int nk_all = (p.K + BK - 1) / BK;
  const int z = blockIdx.z;
  const int kt_begin = (nk_all * z) / gridDim.z;
  const int kt_end = (nk_all * (z + 1)) / gridDim.z;
  const int nk = kt_end - kt_begin;

  const T* A = static_cast<const T*>(p.A);
  // This wave's 32-row weight blocks: block b = n_tile*NB + wid*TN + tn is sub-block
  // b%4 of 128-row group b/4 (rows past N are zero padding of the packed layout; a
  // group past the last one is clamped to it, and the columns it computes are never
  // stored).
  const int n_groups = (p.N + 127) >> 7;
  const T* Bw[TN];
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    const int blk = n_tile * NB + wid * TN + tn;
    const int grp = min(blk >> 2, n_groups - 1);
    Bw[tn] = static_cast<const T*>(p.B) +
             (int64_t(grp) * (p.K >> 4) * 4 + (blk & 3)) * 512 + lane * 8;
  }

  // Argmax tiles compute the transposed product (the weights as the A operand): a lane
  // then holds 16 columns of one row per 32-column block, and the row maxima are taken
  // in registers.  Every other tile holds C = A.W^T (a lane: one column, 16 rows).
  auto mma = [](bf16x8_t act, bf16x8_t w, f32x16_t c) {
    if constexpr (EPI == kEpiArgmax)
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, act, c, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(act, w, c, 0, 0, 0);
  };
  auto mma_f32 = [](float act, float w, f32x16_t c) {
    if constexpr (EPI == kEpiArgmax)
      return __builtin_amdgcn_mfma_f32_32x32x2f32(w, act, c, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f32_32x32x2f32(act, w, c, 0, 0, 0);
  };
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][tn][r] = 0.f;

  if (nk > 0) {
    u32x4 ra[STAGES][A_CH];
    u32x4 rb[STAGES][TN * 4];
    // Activation chunk c of a K-step: row c/8, 16-byte column c%8.  Rows past M are
    // clamped (their products are never stored); loads stay unpredicated so the
    // compiler's outstanding-load counting is exact.
    // In fp32 a last step may have only 16 of its 32 K: the chunks past K repeat the row's
    // last one here and become zeros on their way into LDS, so that whatever finite weight
    // they meet (a clamped block) adds nothing.
    auto load_a = [&](int kt, u32x4* dst) {
      const int64_t k = int64_t(kt_begin + min(kt, nk - 1)) * BK;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int c = min(tid + i * THREADS, A_CHUNKS - 1);   // spare threads repeat the last
        const int row = min(m0 + (c >> 3), p.M - 1);
        const int64_t kc = k + (c & 7) * VEC;
        dst[i] = ld16(A + int64_t(row) * p.lda + (F32 ? min(kc, int64_t(p.K - VEC)) : kc));
      }
    };
    // The ring issues STAGES steps past the last one; those are never used.  Their loads
    // read the activations' first 16 bytes (one line, in L2) rather than the last weight
    // step again: a re-read of the weights would come from HBM (the non-temporal streams
    // do not keep them in L2), STAGES of the nk steps extra (O/down: 2 of 8).  The loads
    // are still issued, so the compiler's outstanding-load counting stays exact.
    auto load_b = [&](int kt, u32x4* dst) {
      const bool live = kt < nk;
      const int64_t kb = int64_t(kt_begin + (live ? kt : 0)) * (BK / 16);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          const T* w = F32 ? Bw[tn] + min(kb + (q >> 1), int64_t(p.K / 16 - 1)) * 4 * 512 + (q & 1) * VEC
                           : Bw[tn] + (kb + q) * 4 * 512;
          const T* src = live ? w : A;
          dst[q * TN + tn] = NT ? ld_nt16(src) : ld16(src);
        }
    };
    auto store_a = [&](const u32x4* src, int kt, int buf) {
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int c = min(tid + i * THREADS, A_CHUNKS - 1);
        const bool in = !F32 || (kt_begin + kt) * BK + (c & 7) * VEC < p.K;
        *reinterpret_cast<u32x4*>(&As[buf][c >> 3][(c & 7) * VEC]) = in ? src[i] : u32x4{0, 0, 0, 0};
      }
    };
    const int arow = lane & 31;
    const int kof = 8 * (lane >> 5);
    auto compute = [&](int buf, const u32x4* bq) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (F32) {   // four of the eight values of 16-K block q/2
          u32x4 af[TM];
#pragma unroll
          for (int i = 0; i < TM; ++i)
            af[i] = *reinterpret_cast<const u32x4*>(
                &As[buf][arow + 32 * i][(q >> 1) * 16 + kof + (q & 1) * VEC]);
#pragma unroll
          for (int e = 0; e < VEC; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int tn = 0; tn < TN; ++tn)
                acc[i][tn] = mma_f32(__uint_as_float(af[i][e]), __uint_as_float(bq[q * TN + tn][e]),
                                     acc[i][tn]);
        } else {
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const bf16x8_t af =
                *reinterpret_cast<const bf16x8_t*>(&As[buf][arow + 32 * i][q * 16 + kof]);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
              acc[i][tn] = mma(af, __builtin_bit_cast(bf16x8_t, bq[q * TN + tn]), acc[i][tn]);
          }
        }
      }
    };
    // Prologue.  The weights do not depend on the previous kernel, so B(0) is issued first
    // and its HBM latency overlaps the activations' L2 latency (issued after A(0) it came
    // one L2 round trip later).  Then A(1..STAGES-1) and B(1..STAGES-1) in the order they
    // are consumed, A(0) into LDS (loads complete in issue order: this waits for B(0) and
    // A(0) only), and A(STAGES) into the register slot A(0) leaves.
    load_b(0, rb[0]);
    load_a(0, ra[0]);
#pragma unroll
    for (int st = 1; st < STAGES; ++st) {
      load_a(st, ra[st]);
      load_b(st, rb[st]);
    }
    store_a(ra[0], 0, 0);
    load_a(STAGES, ra[0]);
    __syncthreads();
    // Step t (ring slot u = t % STAGES): compute with A(t) in LDS and B(t) in rb[u];
    // move A(t+1) into the other LDS buffer; refill the freed slots with A(t+1+STAGES)
    // and B(t+STAGES); barrier.
    auto step = [&](int t, int u) {
      compute(t & 1, rb[u]);
      store_a(ra[(u + 1) % STAGES], t + 1, (t + 1) & 1);
      load_a(t + 1 + STAGES, ra[(u + 1) % STAGES]);
      load_b(t + STAGES, rb[u]);
      __syncthreads();
    };
    int kt = 0;
    for (; kt + STAGES <= nk; kt += STAGES) {
#pragma unroll
      for (int u = 0; u < STAGES; ++u) step(kt + u, u);
    }
#pragma unroll
    for (int u = 0; u < STAGES; ++u)
      if (kt + u < nk) step(kt + u, u);
  }

  if constexpr (EPI == kEpiPartial) {
    float* C = p.C + int64_t(z) * p.M * p.N;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int col = n0 + 32 * (wid * TN + tn) + (lane & 31);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (row < p.M && col < p.N) C[int64_t(row) * p.N + col] = acc[i][tn][r];
        }
    }
  } else {
    // Transposed tile: lane l holds row 32i + l%32 and, of 32-column block b, columns
    // 32b + 8(r/4) + 4(l/32) + r%4 (r = 0..15).  Each lane scans its columns in increasing
    // order (lowest column on ties), the two lane halves of a row meet by a shuffle, the
    // waves' (max, column) pairs meet in LDS, and one atomic per row folds the tile's pair
    // into the row's packed key.  The K loop ended with a barrier, so LDS is free.
    float* Cs = reinterpret_cast<float*>(smem);
    const int tok = lane & 31;
    float best[TM];
    int bcol[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      best[i] = -INFINITY;
      bcol[i] = 0x7FFFFFFF;
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int cb = n0 + 32 * (wid * TN + tn) + 4 * (lane >> 5);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int col = cb + 8 * (r >> 2) + (r & 3);
        const bool in = col < p.N;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          // selects, not branches: one compare and two conditional moves per value
          const float v = acc[i][tn][r];
          const bool take = in & (v > best[i]);
          best[i] = take ? v : best[i];
          bcol[i] = take ? col : bcol[i];
        }
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
    if (p.C != nullptr) {
      // Logits (tests, sampling): the tile goes through LDS four waves (128 columns) at a
      // time ([block][row][column of the block]) and leaves as coalesced rows.
#pragma unroll
      for (int slab = 0; slab < NB / 4; ++slab) {
        if (slab > 0) __syncthreads();
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          const int b = wid * TN + tn;
          if ((b >> 2) == slab) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int r = 0; r < 16; ++r)
                Cs[((b & 3) * BM + 32 * i + tok) * LDC + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] =
                    acc[i][tn][r];
          }
        }
        __syncthreads();
        const int cs0 = n0 + 128 * slab;
        for (int e = tid; e < BM * 128; e += THREADS) {
          const int rr = e >> 7, cc = e & 127;
          if (m0 + rr < p.M && cs0 + cc < p.N)
            p.C[int64_t(m0 + rr) * p.N + cs0 + cc] = Cs[((cc >> 5) * BM + rr) * LDC + (cc & 31)];
        }
      }
      __syncthreads();
    }
    float* rv = Cs;                                          // [wave][row] maxima
    int* rc = reinterpret_cast<int*>(Cs + NW * BM);          // [wave][row] columns
    if (lane < 32) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        rv[wid * BM + 32 * i + tok] = best[i];
        rc[wid * BM + 32 * i + tok] = bcol[i];
      }
    }
    __syncthreads();
    if (tid < BM && m0 + tid < p.M) {
      float bv = rv[tid];
      int bc = rc[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float ov = rv[w * BM + tid];
        const int oc = rc[w * BM + tid];
        if (ov > bv || (ov == bv && oc < bc)) {
          bv = ov;
          bc = oc;
        }
      }
      if (bc != 0x7FFFFFFF) atomicMax(p.keys + m0 + tid, argmax_key(bv, bc));
    }
  }
}

__global__ void argmax_finalize_kernel(unsigned long long* keys, int64_t M, int32_t* argmax,
                                       float* max_logit) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= M) return;
  decode_argmax_key(keys[i], argmax + i, max_logit != nullptr ? max_logit + i : nullptr);
  keys[i] = 0ull;   // the workspace is handed back zeroed
}

// Row-major [N][K] -> packed layout, one 16-byte (bf16) or 32-byte (fp32) lane chunk
// of 8 elements per thread; rows N..ceil(N/128)*128-1 are written as zeros.
template <typename T>
__global__ void pack_weight_kernel(const T* __restrict__ src, T* __restrict__ dst, int N, int K) {
  const int64_t chunks = int64_t((N + 127) / 128) * (K / 16) * 4 * 64;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < chunks;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int lane = int(e & 63);
    const int64_t blk = e >> 6;                 // ((group * (K/16)) + kb) * 4 + sub
    const int sub = int(blk & 3);
    const int64_t kb = (blk >> 2) % (K / 16), grp = (blk >> 2) / (K / 16);
    const int64_t n = grp * 128 + sub * 32 + (lane & 31);
    const int64_t k = kb * 16 + 8 * (lane >> 5);
    T* d = dst + e * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] = (n < N) ? src[n * K + k + j] : T(0);
  }
}

// ---------------------------------------------------------------------------- host side

template <int NW, int STAGES, bool NT>
static void launch_bf16_partial(const GemmArgs& a, int splits, hipStream_t s) {
  constexpr int TN = 1;
  const int BM = (a.M <= 64 && a.M2 <= 64) ? 64 : 128;
  constexpr int BN = 32 * NW * TN;
  const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) +
                    ((a.M2 + BM - 1) / BM) * ((a.N2 + BN - 1) / BN);
  const dim3 grid(tiles, 1, splits), block(NW * 64);
  if (BM == 64)
    hipLaunchKernelGGL((gemm_kernel<bf16_t, 64, NW, STAGES, kEpiPartial, TN, NT>), grid, block, 0, s,
                       a);
  else
    hipLaunchKernelGGL((gemm_kernel<bf16_t, 128, NW, STAGES, kEpiPartial, TN, NT>), grid, block, 0, s,
                       a);
}

// One pass for 128 < M <= 192 rows: every row in one tile, 8 waves of one 32-column block,
// the weights streamed once (non-temporal).  In turns with the matrix-core bound tiles, which pad
// the rows to 256, 129280 columns of 4096: 192 rows 217 us here, 193 rows 227 there (32000
// columns, 125 workgroups of either: 76 and 78).  Above 192 rows those are the faster ones (208
// rows 234-239 against 266 us for one tile of 256 rows, whose activation fragments are the LDS
// bandwidth of the CU).
static void launch_bf16_argmax_tall(const GemmArgs& a, hipStream_t s) {
  constexpr int BN = 32 * 8;
  const dim3 grid((a.N + BN - 1) / BN, 1, 1), block(8 * 64);
  hipLaunchKernelGGL((gemm_kernel<bf16_t, 192, 8, 2, kEpiArgmax, 1, true>), grid, block, 0, s, a);
}

// Up to 128 rows: one row tile, every weight byte is read once, so the weights stream past the
// caches.
template <int BM, int NW, int TN, int STAGES>
static void launch_bf16_argmax_stream(const GemmArgs& a, hipStream_t s) {
  constexpr int BN = 32 * NW * TN;
  hipLaunchKernelGGL((gemm_kernel<bf16_t, BM, NW, STAGES, kEpiArgmax, TN, true>),
                     dim3((a.N + BN - 1) / BN), dim3(NW * 64), 0, s, a);
}

// The narrowest tile that covers the vocabulary in one round of workgroups: 128, 256 or 512
// columns.  Wider ones leave CUs without a stream (4096-wide states, 64 rows: 32000 columns
// 88 us in 512-column tiles, 55 in 256, 42 in 128; 50000 columns 93, 62, 71; 64000 columns 98,
// 77, 88), narrower ones take a second round and re-read the activations more often (100000
// columns 121, 129, 142).  Ring depths as measured at each width.
static void launch_bf16_argmax(const GemmArgs& a, hipStream_t s) {
  const int ncu = device_cu_count();
  const bool low = a.M <= 64;
  if ((int64_t(a.N) + 127) / 128 <= ncu)
    low ? launch_bf16_argmax_stream<64, 4, 1, 4>(a, s) : launch_bf16_argmax_stream<128, 4, 1, 2>(a, s);
  else if ((int64_t(a.N) + 255) / 256 <= ncu)
    low ? launch_bf16_argmax_stream<64, 8, 1, 2>(a, s) : launch_bf16_argmax_stream<128, 8, 1, 2>(a, s);
  else
    low ? launch_bf16_argmax_stream<64, 8, 2, 2>(a, s) : launch_bf16_argmax_stream<128, 8, 2, 2>(a, s);
}

// fp32 tiles: 4 waves of one 32-column block and 32, 64 or 128 rows (the plan's tn row
// blocks), bound by the fp32 matrix rate from about 64 rows (a 32 x 16 weight block is 2 KB
// against 512 matrix-core cycles per 32 rows) and by the weight stream below.  One row tile
// streams its weights past the caches.  64 rows: projections of K = 1024-4096 44 -> 12.6 us
// (median of five shapes), the 1024 x 32000 head 249 -> 53 us against 64 x 64 tiles on the
// vector units.
template <int EPI, int BM, int STAGES>
static void launch_f32(const GemmArgs& a, int splits, hipStream_t s) {
  const int mt = (a.M + BM - 1) / BM;
  const dim3 grid(mt * ((a.N + 127) / 128), 1, splits), block(256);
  if (mt == 1)
    hipLaunchKernelGGL((gemm_kernel<float, BM, 4, STAGES, EPI, 1, true>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((gemm_kernel<float, BM, 4, STAGES, EPI, 1, false>), grid, block, 0, s, a);
}

template <int EPI>
static void launch_f32(const GemmArgs& a, const GemmPlan& plan, hipStream_t s) {
  if (plan.tn == 1)
    launch_f32<EPI, 32, 4>(a, plan.splits, s);
  else if (plan.tn == 2)
    launch_f32<EPI, 64, 3>(a, plan.splits, s);
  else
    launch_f32<EPI, 128, 2>(a, plan.splits, s);
}

// Rows of a tile and K splits of an fp32 problem.  A workgroup's products take 32 cycles per
// 32 rows and unit of K on each SIMD (the fp32 matrix rate); tiles of 32 rows run 7% and tiles
// of 128 rows 3% off the 64-row ones' pace at equal rows (128 rows x 1024 -> 32000: 77, 72 and
// 78 us), so the smaller tile wins where it pads fewer rows (65 rows: 59, 72, 78) or gives idle
// CUs a workgroup (64 rows -> 4000: 24 against 40 us).  Every split writes and the next kernel
// reads an fp32 partial (about 1700 B a cycle over the chip); a split keeps two K steps.
static GemmPlan f32_plan(int M, int N, int K, int max_splits) {
  const int ncu = device_cu_count();
  const int steps = (K + kBKf32 - 1) / kBKf32;
  GemmPlan best{4, 1, 1};
  double best_t = 1e30;
  for (int tn : {2, 1, 4}) {
    const int BM = 32 * tn;
    const int64_t tiles = ((int64_t(M) + BM - 1) / BM) * ((N + 127) / 128);
    const double pace = tn == 1 ? 1.07 : tn == 2 ? 1.0 : 1.03;
    const double part = max_splits > 1 ? double(M) * N * 8.0 / 1700.0 : 0.0;
    for (int sp = 1; sp <= max_splits && (sp == 1 || steps / sp >= 2) && sp * part < best_t; ++sp) {
      const double mma = double((tiles * sp + ncu - 1) / ncu) * ((steps + sp - 1) / sp) * BM * kBKf32 * pace;
      const double t = mma + sp * part;
      if (t < best_t * (1.0 - 1e-9)) {
        best_t = t;
        best = GemmPlan{4, sp, tn};
      }
    }
  }
  return best;
}

static hipError_t launch_gemm_any(bool bf16, int epi, const GemmArgs& a, GemmPlan plan,
                                  hipStream_t s) {
  if (bf16) {
    if (epi == kEpiPartial) {
      if (plan.tn > 1) return launch_gemm_deep(kEpiPartial, a, plan, s);
      if (!plan.nt && plan.nw == 4) {
        launch_bf16_partial<4, 4, false>(a, plan.splits, s);
      } else if (!plan.nt) {
        launch_bf16_partial<8, 4, false>(a, plan.splits, s);
      } else if (plan.nw == 8) {
        launch_bf16_partial<8, 4, true>(a, plan.splits, s);
      } else if (plan.nw == 6) {
        launch_bf16_partial<6, 3, true>(a, plan.splits, s);
      } else {
        launch_bf16_partial<4, 2, true>(a, plan.splits, s);
      }
    } else {
      if (a.M > 192) return launch_gemm_deep(kEpiArgmax, a, deep_argmax_plan(a.M), s);
      if (a.M > 128)
        launch_bf16_argmax_tall(a, s);
      else
        launch_bf16_argmax(a, s);
    }
    return hipGetLastError();
  }
  if (epi == kEpiPartial)
    launch_f32<kEpiPartial>(a, plan, s);
  else
    launch_f32<kEpiArgmax>(a, f32_plan(a.M, a.N, a.K, 1), s);
  return hipGetLastError();
}

int gemm_k_align(bool bf16) { return bf16 ? kBK : 16; }

GemmPlan gemm_plan(bool bf16, int M, int N, int K) { return gemm_plan2(bf16, M, N, 0, 0, K); }

static GemmPlan plan_stream(int BM, int M, int N, int M2, int N2, int nk, int ncu,
                            std::initializer_list<int> waves);

GemmPlan gemm_plan2(bool bf16, int M, int N, int M2, int N2, int K) {
  const int ncu = device_cu_count();
  if (!bf16) return f32_plan(M, N, K, kMaxSplits);
  const int nk = K / kBK;
  // One workgroup per CU works best for these weight streams: a CU holding two
  // workgroups while others hold one doubles the kernel's critical path.  Pick the
  // tile width (4, 6 or 8 waves of 32 columns) and K split whose workgroup count fills
  // the CUs best without exceeding them; ties go to fewer splits (less partial
  // traffic) and then to more waves (more bytes in flight per CU).  Every split keeps
  // at least 8 K-steps.
  // Above 128 rows the products are matrix-core bound (gemm_deep.hip).
  const int BM = (M <= 64 && M2 <= 64) ? 64 : 128;
  if (M > 128 || M2 > 128) return deep_plan(M, N, M2, N2, K);
  return plan_stream(BM, M, N, M2, N2, nk, ncu, {4, 6, 8});
}

GemmPlan gemm_plan_shared(int M, int N, int M2, int N2, int K) {
  // The row tiles of the first problem (at most two) read the same weight columns at
  // about the same time on one XCD: 8-wave tiles with the weights fetched through L2, or 4-wave
  // ones where they fill the CUs as well or better, up to K = 4096.  Two-layer drafters (d_ff =
  // 2d) of 4 x 16 block rows, 4 and 8 waves offered against 8: d = 2304 153 us against 156,
  // 2560 163.5 / 166.5, 3072 188 / 192, 3584 217 / 218.5; beyond, where half the weight bytes
  // in flight cost more than the fill gives, 5120 335 / 328 and with 8 x 16 rows 425 / 419, 6144
  // 526.5 / 521.  (Short K takes 4 waves: 64 + 64 rows x 1024 -> 3072 48 workgroups in place of
  // 24, the two-layer step 150.9 -> 147.3 us.)
  const int nk = K / kBK, ncu = device_cu_count();
  GemmPlan p = K <= 4096 ? plan_stream(128, M, N, M2, N2, nk, ncu, {4, 8})
                         : plan_stream(128, M, N, M2, N2, nk, ncu, {8});
  p.nt = false;
  return p;
}

static GemmPlan plan_stream(int BM, int M, int N, int M2, int N2, int nk, int ncu,
                            std::initializer_list<int> waves) {
  const int tn = 1;
  if (nk <= kShortSteps) {
    // Short K: the launch is a chain of K steps (0.22 us each at 64 rows, 0.35 at 128) and the
    // partials that each split adds (3.8 TB/s written and read back); the narrowest tiles and
    // the split with the least sum, in one round and with three steps at least.
    const int tiles = ((M + BM - 1) / BM) * ((N + 127) / 128) + ((M2 + BM - 1) / BM) * ((N2 + 127) / 128);
    if (tiles <= ncu) {
      const double step = BM == 64 ? 0.22 : 0.35;
      const double part = (double(M) * N + double(M2) * N2) * 8.0 / 3.8e6;
      int best_s = 1;
      double best_t = 1e30;
      for (int s = 1; s <= kMaxSplits && tiles * s <= ncu && (s == 1 || nk / s >= 3); ++s) {
        const double t = step * ((nk + s - 1) / s) + part * s;
        if (t < best_t) {
          best_t = t;
          best_s = s;
        }
      }
      return GemmPlan{4, best_s, tn};
    }
  }
  GemmPlan best{4, 1, tn};
  double best_fill = -1.0;
  for (int nw : waves) {
    const int bn = 32 * nw * tn;
    const int tiles = ((M + BM - 1) / BM) * ((N + bn - 1) / bn) +
                      ((M2 + BM - 1) / BM) * ((N2 + bn - 1) / bn);
    for (int s = 1; s <= kMaxSplits; ++s) {
      if (s > 1 && nk / s < 8) break;
      const int wgs = tiles * s;
      const int rounds = (wgs + ncu - 1) / ncu;
      const double fill = double(wgs) / double(rounds * ncu);   // busy fraction of CU-rounds
      // Prefer a single round; more rounds only when they are nearly full.
      const double score = fill / rounds + (rounds == 1 ? 1.0 : 0.0);
      const bool tie = score > best_fill - 1e-9 && score < best_fill + 1e-9;
      if (score > best_fill + 1e-9 ||
          (tie && (s < best.splits || (s == best.splits && nw > best.nw)))) {
        best_fill = score;
        best = GemmPlan{nw, s, tn};
      }
    }
  }
  return best;
}

size_t packed_weight_elems(int N, int K) { return size_t((N + 127) / 128) * 128 * size_t(K); }

hipError_t launch_pack_weight(bool bf16, const void* src, void* dst, int N, int K, hipStream_t s) {
  const int64_t chunks = int64_t((N + 127) / 128) * (K / 16) * 4 * 64;
  int64_t blocks = (chunks + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) return hipSuccess;
  if (bf16)
    hipLaunchKernelGGL(pack_weight_kernel<bf16_t>, dim3(unsigned(blocks)), dim3(256), 0, s,
                       static_cast<const bf16_t*>(src), static_cast<bf16_t*>(dst), N, K);
  else
    hipLaunchKernelGGL(pack_weight_kernel<float>, dim3(unsigned(blocks)), dim3(256), 0, s,
                       static_cast<const float*>(src), static_cast<float*>(dst), N, K);
  return hipGetLastError();
}

hipError_t launch_gemm_partial(bool bf16, const void* A, int64_t lda, const void* B, int M, int N,
                               int K, GemmPlan plan, float* C, hipStream_t s) {
  GemmArgs a{};
  a.A = A; a.lda = lda; a.B = B;
  a.M = M; a.N = N; a.K = K; a.C = C; a.keys = nullptr;
  return launch_gemm_any(bf16, kEpiPartial, a, plan, s);
}

hipError_t launch_gemm_partial2(const void* A, int64_t lda, const void* B, int M, int N,
                                float* C, const void* A2, int64_t lda2, const void* B2, int M2,
                                int N2, float* C2, int K, GemmPlan plan, hipStream_t s) {
  GemmArgs a{};
  a.A = A; a.lda = lda; a.B = B;
  a.M = M; a.N = N; a.K = K; a.C = C; a.keys = nullptr;
  a.A2 = A2; a.lda2 = lda2; a.B2 = B2; a.M2 = M2; a.N2 = N2; a.C2 = C2;
  return launch_gemm_any(true, kEpiPartial, a, plan, s);
}

hipError_t launch_gemm_rows(const void* A, int64_t lda, const void* B, int M, int N, int K,
                            GemmPlan plan, const float* bias, void* out, hipStream_t s) {
  if (plan.tn < 2 || plan.splits != 1 || N % 8 != 0) return hipErrorInvalidValue;
  GemmArgs a{};
  a.A = A; a.lda = lda; a.B = B;
  a.M = M; a.N = N; a.K = K; a.out = out; a.bias = bias;
  return launch_gemm_deep(kEpiRows, a, plan, s);
}

bool gemm_gated_plan(int M, int F, int K, GemmPlan* plan) {
  return M > 128 && F % 64 == 0 && deep_gated_plan(M, F, K, plan);
}

hipError_t launch_gemm_gated(const void* A, int64_t lda, const void* W, int M, int F, int K,
                             GemmPlan plan, void* act, hipStream_t s) {
  if (plan.tn < 2 || plan.splits != 1 || F % 64 != 0) return hipErrorInvalidValue;
  GemmArgs a{};
  a.A = A; a.lda = lda; a.B = W;
  a.M = M; a.N = 2 * F; a.K = K; a.out = act;
  return launch_gemm_deep(kEpiGated, a, plan, s);
}

hipError_t launch_gemm_kv(const void* A, int64_t lda, const void* B, int M, int d, int hd,
                          GemmPlan plan, const int32_t* plan_pos, const int32_t* plan_row,
                          const float* rope_cs, void* kc, void* vtc, int64_t cap, hipStream_t s) {
  // 512-column tiles lie wholly in K or in V when d % 512 == 0.
  if (plan.tn < 2 || plan.splits != 1 || (hd != 64 && hd != 128) || d % 512 != 0)
    return hipErrorInvalidValue;
  if (M <= 0) return hipSuccess;
  GemmArgs a{};
  a.A = A; a.lda = lda; a.B = B;
  a.M = M; a.N = 2 * d; a.K = d;
  a.plan_pos = plan_pos; a.plan_row = plan_row; a.rope_cs = rope_cs;
  a.kc = kc; a.vtc = vtc; a.cap = cap; a.kv_d = d; a.hd = hd;
  return launch_gemm_deep(kEpiKV, a, plan, s);
}

hipError_t launch_lm_head_keys(bool bf16, const void* hidden, const void* W, int64_t M, int d,
                               int V, unsigned long long* keys, float* logits, hipStream_t s) {
  // keys are zero on entry (the workspace contract); the GEMM folds every row's maximum
  // into them.  Rows are processed in chunks that keep the int32 tile arithmetic in range.
  const int64_t chunk = 1 << 20;
  for (int64_t r0 = 0; r0 < M; r0 += chunk) {
    const int rows = int(M - r0 < chunk ? M - r0 : chunk);
    GemmArgs a{};
    const size_t el = bf16 ? 2 : 4;
    a.A = static_cast<const char*>(hidden) + r0 * d * el;
    a.lda = d; a.B = W;
    a.M = rows; a.N = V; a.K = d;
    a.C = logits != nullptr ? logits + r0 * V : nullptr;
    a.keys = keys + r0;
    const hipError_t e = launch_gemm_any(bf16, kEpiArgmax, a, GemmPlan{}, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_lm_head(bool bf16, const void* hidden, const void* W, int64_t M, int d, int V,
                          unsigned long long* keys, int32_t* argmax, float* max_logit,
                          float* logits, hipStream_t s) {
  const hipError_t e = launch_lm_head_keys(bf16, hidden, W, M, d, V, keys, logits, s);
  if (e != hipSuccess) return e;
  // The finalize pass turns the keys into outputs and clears them.
  const int threads = 256;
  const unsigned blocks = unsigned((M + threads - 1) / threads);
  hipLaunchKernelGGL(argmax_finalize_kernel, dim3(blocks), dim3(threads), 0, s, keys, M, argmax,
                     max_logit);
  return hipGetLastError();
}

}  // namespace hdf
