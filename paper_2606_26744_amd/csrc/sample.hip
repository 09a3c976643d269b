// Temperature sampling of draft tokens and speculative-sampling verification (the
// temperature-1 results of the paper's tables; the rule itself is the standard one of
// speculative decoding, which the paper does not restate: accept draft x_i with
// probability min(1, p_i(x_i) / q_i(x_i)), at the first rejection draw from
// max(0, p - q) renormalised, after K acceptances draw the bonus from p_K).
//
// Random numbers: Philox4x64-10 (Salmon et al., SC'11), key (seed, stream), counter
// (row, v/8, purpose, 0); word (v%8)/2 of the block gives two uniforms, from its high
// 32 bits for even v and its low 32 bits for odd v: u = (top 24 bits + 1/2) * 2^-24.  A draw from
// softmax(s) is argmax_v (s_v - log(-log u_v)) (Gumbel-max), so no probability vector
// is ever materialised: a pass over the logits keeps a running log-sum-exp and the
// best perturbed score.
#include "common.hpp"
#include "kernels.hpp"

namespace hdf {

constexpr int kSampleThreads = 256;
constexpr int kPurposeDraft = 0, kPurposeAccept = 1, kPurposeResample = 2;

// 64 x 64 -> 128 bits from four 32 x 32 -> 64 products, on 32-bit halves: a half that every
// lane shares (the row, the purpose and what the first rounds make of them) stays on the
// scalar unit and so do the products of two such halves.
struct U128 {
  uint32_t w[4];
};
__device__ __forceinline__ U128 mul_64x64(uint32_t a0, uint32_t a1, uint64_t b) {
  const uint32_t b0 = uint32_t(b), b1 = uint32_t(b >> 32);
  const uint64_t p0 = uint64_t(a0) * b0;
  const uint64_t p1 = uint64_t(a0) * b1 + (p0 >> 32);
  const uint64_t p2 = uint64_t(a1) * b0 + uint32_t(p1);
  const uint64_t p3 = uint64_t(a1) * b1 + (p1 >> 32) + (p2 >> 32);
  return {{uint32_t(p0), uint32_t(p2), uint32_t(p3), uint32_t(p3 >> 32)}};
}

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1) {
  uint32_t v[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[2 * j] = uint32_t(c[j]);
    v[2 * j + 1] = uint32_t(c[j] >> 32);
  }
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B97F4A7C15ull;
      k1 += 0xBB67AE8584CAA73Bull;
    }
    const U128 x = mul_64x64(v[0], v[1], 0xD2E7470EE14C6C93ull);
    const U128 y = mul_64x64(v[4], v[5], 0xCA5A826395121157ull);
    const uint32_t n0 = y.w[2] ^ v[2] ^ uint32_t(k0), n1 = y.w[3] ^ v[3] ^ uint32_t(k0 >> 32);
    const uint32_t n4 = x.w[2] ^ v[6] ^ uint32_t(k1), n5 = x.w[3] ^ v[7] ^ uint32_t(k1 >> 32);
    v[0] = n0; v[1] = n1; v[2] = y.w[0]; v[3] = y.w[1];
    v[4] = n4; v[5] = n5; v[6] = x.w[0]; v[7] = x.w[1];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = uint64_t(v[2 * j]) | (uint64_t(v[2 * j + 1]) << 32);
}

// The 24-bit draws k of the eight entries 8*g .. 8*g+7 of one row; entry uniform u = (k + 1/2) / 2^24.
__device__ __forceinline__ void draws8(uint64_t seed, uint64_t stream, uint64_t row, uint64_t g,
                                       int purpose, uint32_t k[8]) {
  uint64_t c[4] = {row, g, uint64_t(purpose), 0ull};
  philox4x64_10(c, seed, stream);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    k[2 * j] = uint32_t(c[j] >> 40);
    k[2 * j + 1] = uint32_t(c[j] & 0xFFFFFFFFull) >> 8;
  }
}

// u rounded to fp32: up to 2^-25 off, and 1 for the greatest.
__device__ __forceinline__ float uniform(uint32_t k) {
  return (float(k) + 0.5f) * 5.9604644775390625e-8f;
}
// -log2(u).  The rounding of k + 1/2 (from 2^23 on) would change it by up to 2^-25 / (1 - u) of
// itself, a third at the greatest uniforms and all of it at the last, whose column would win the
// draw whatever its probability: what the sum lost is taken off to first order.
__device__ __forceinline__ float neg_log2_uniform(uint32_t k) {
  const float a = float(k), s = a + 0.5f;
  const float lost = (a - s) + 0.5f;   // exact: 0 or +-1/2
  return fmaf(lost, -8.5991325e-8f, fabsf(__builtin_amdgcn_logf(s * 5.9604644775390625e-8f)));
}

constexpr int kGroupsPerPass = 4;   // 8-entry groups each thread loads before computing

// The draw as a race: argmax_v (s_v - log(-log u_v)) is argmax_v e^(s_v - m) / -log2(u_v)
// for any m, so the entries compare by this ratio, whose numerator the log-sum-exp needs
// anyway, and only a thread's winner takes a logarithm of it.
__device__ __forceinline__ float race(float p, uint32_t k) {
  return p * __builtin_amdgcn_rcpf(neg_log2_uniform(k));
}
// Perturbed score s_v - log(-log u_v) of a ratio with numerator e^(s_v - m).
__device__ __forceinline__ float race_score(float ratio, float m) {
  return m + (logf(ratio) + 0.36651292058166435f);   // - log(log 2)
}

__device__ __forceinline__ unsigned long long sample_key(float score, int v) {
  return (static_cast<unsigned long long>(f32_order_key(score)) << 32) |
         static_cast<unsigned long long>(0xFFFFFFFFu - static_cast<uint32_t>(v));
}

// Running state of one thread over part of a row: log-sum-exp (m, s) of the scaled
// logits and the best perturbed score (ties to the lowest index).
struct RowState {
  float m, s, best;
  int idx;
};

__device__ __forceinline__ void merge(RowState& a, const RowState& b) {
  if (b.s > 0.f) {
    if (a.s == 0.f) {
      a.m = b.m;
      a.s = b.s;
    } else if (b.m > a.m) {
      a.s = a.s * __expf(a.m - b.m) + b.s;
      a.m = b.m;
    } else {
      a.s += b.s * __expf(b.m - a.m);
    }
  }
  if (b.best > a.best || (b.best == a.best && b.idx < a.idx)) {
    a.best = b.best;
    a.idx = b.idx;
  }
}

// Workgroup reduction of RowState (all threads get the result).
__device__ RowState block_merge(RowState st, RowState* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    RowState b;
    b.m = __shfl_xor(st.m, o, kWave);
    b.s = __shfl_xor(st.s, o, kWave);
    b.best = __shfl_xor(st.best, o, kWave);
    b.idx = __shfl_xor(st.idx, o, kWave);
    merge(st, b);
  }
  if (lane == 0) sh[wid] = st;
  __syncthreads();
  RowState t = sh[0];
  for (int w = 1; w < int(blockDim.x >> 6); ++w) merge(t, sh[w]);
  __syncthreads();
  return t;
}

// The drawing pass is bound by the vector unit's integer products (a Philox block of eight
// uniforms is about 62 32-bit products after the shared halves are taken out), not by its
// 16-byte loads: 128 rows x 129280, 43.6 -> 31.7 us with 32-bit halves in the generator and
// the race in place of two logarithms an entry, 32.8 with the uniforms' rounding taken off.  The
// pass without draws streams the rows (14.7 us, 4.5 TB/s).
// Pass over logits row `row`, columns [c0, c1) (c0 % 8 == 0): partial log-sum-exp of
// logits * inv_t and, with SAMPLE, the Gumbel-max draw.  Partial j of the row goes to
// part[row * n_parts + j].  Each thread loads kGroupsPerPass groups of eight logits
// (two 16-byte loads each when the row is 16-byte aligned) before it computes, so that
// the loads of a pass are in flight together.
template <bool SAMPLE>
__global__ void __launch_bounds__(kSampleThreads)
row_pass_kernel(const float* __restrict__ logits, int64_t ld, int V, int n_parts, int chunk,
                float inv_t, uint64_t seed, uint64_t stream, RowState* __restrict__ part) {
  __shared__ RowState sh[kSampleThreads / 64];
  const int64_t row = blockIdx.x;
  const int j = blockIdx.y;
  const int c0 = j * chunk, c1 = min(V, c0 + chunk);
  const float* z = logits + row * ld;
  const bool vec = (reinterpret_cast<uintptr_t>(z) & 15u) == 0;
  RowState st{-INFINITY, 0.f, -INFINITY, 0x7FFFFFFF};
  float ratio = 0.f;   // best ratio so far, numerators relative to st.m
  for (int g0 = c0 / 8 + threadIdx.x; 8 * g0 < c1; g0 += kSampleThreads * kGroupsPerPass) {
    float x[kGroupsPerPass][8];
#pragma unroll
    for (int q = 0; q < kGroupsPerPass; ++q) {
      const int v0 = 8 * (g0 + q * kSampleThreads);
      if (vec && v0 + 8 <= c1) {
        const float4 a = *reinterpret_cast<const float4*>(z + v0);
        const float4 b = *reinterpret_cast<const float4*>(z + v0 + 4);
        x[q][0] = a.x; x[q][1] = a.y; x[q][2] = a.z; x[q][3] = a.w;
        x[q][4] = b.x; x[q][5] = b.y; x[q][6] = b.z; x[q][7] = b.w;
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) x[q][k] = (v0 + k < c1) ? z[v0 + k] : 0.f;
      }
    }
#pragma unroll
    for (int q = 0; q < kGroupsPerPass; ++q) {
      const int g = g0 + q * kSampleThreads;
      if (8 * g >= c1) continue;
      const int nv = min(8, c1 - 8 * g);   // valid entries of the group (8 but at the end)
      float xs[8];
      float gm = -INFINITY;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        xs[k] = k < nv ? x[q][k] * inv_t : -INFINITY;
        gm = fmaxf(gm, xs[k]);
      }
      // One rescale per group: s <- s e^(m - m') + sum_k e^(x_k - m'), m' = max(m, max_k x_k).
      // While every entry was -inf (masked columns), the exponents refer to 0.
      const float mn = fmaxf(st.m, gm);
      const float ref = mn == -INFINITY ? 0.f : mn;
      float add = 0.f;
      float p[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        p[k] = __expf(xs[k] - ref);
        add += p[k];
      }
      const float down = __expf(st.m - ref);
      st.s = st.s * down + add;
      st.m = mn;
      if constexpr (SAMPLE) {
        uint32_t dr[8];
        draws8(seed, stream, uint64_t(row), uint64_t(g), kPurposeDraft, dr);
        // The group's best ratio, lowest index first (entries past the end have p = 0, the
        // group's largest p = 1 or a running maximum above it); groups come in increasing
        // order, so a tie with the running best keeps the running (lower) index.
        float gb = 0.f;
        int gk = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float r = race(p[k], dr[k]);
          const bool take = r > gb;
          gb = take ? r : gb;
          gk = take ? k : gk;
        }
        if (mn < INFINITY) {
          ratio *= down;
          if (gb > ratio) {
            ratio = gb;
            st.idx = 8 * g + gk;
          }
        } else if (ratio < INFINITY) {
          // A scaled logit beyond fp32 (a temperature near 0): the first one wins, as an
          // infinite score does; its numerator is e^(inf - inf).
#pragma unroll
          for (int k = 7; k >= 0; --k)
            if (p[k] != p[k]) {
              ratio = INFINITY;
              st.idx = 8 * g + k;
            }
        }
      }
    }
  }
  if (st.idx != 0x7FFFFFFF) st.best = race_score(ratio, st.m);
  st = block_merge(st, sh);
  if (threadIdx.x == 0) part[row * n_parts + j] = st;
}

// A row's partials combined by one wave; every lane gets the result.
__device__ __forceinline__ RowState row_combine(const RowState* __restrict__ part, int n_parts) {
  RowState a{-INFINITY, 0.f, -INFINITY, 0x7FFFFFFF};
  for (int j = threadIdx.x & 63; j < n_parts; j += 64) merge(a, part[j]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    RowState b;
    b.m = __shfl_xor(a.m, o, kWave);
    b.s = __shfl_xor(a.s, o, kWave);
    b.best = __shfl_xor(a.best, o, kWave);
    b.idx = __shfl_xor(a.idx, o, kWave);
    merge(a, b);
  }
  return a;
}

// lse[row] = m + log(s); token[row] = best index.  One wave per row.
__global__ void __launch_bounds__(kSampleThreads)
row_finish_kernel(const RowState* __restrict__ part, int64_t rows, int n_parts,
                  float* __restrict__ lse, int32_t* __restrict__ tokens) {
  const int64_t row = int64_t(blockIdx.x) * (kSampleThreads / 64) + (threadIdx.x >> 6);
  if (row >= rows) return;
  const RowState a = row_combine(part + row * n_parts, n_parts);
  if ((threadIdx.x & 63) != 0) return;
  if (lse != nullptr) lse[row] = a.m + logf(a.s);
  if (tokens != nullptr) tokens[row] = a.idx;
}

static void row_split(int64_t rows, int V, int& n_parts, int& chunk) {
  // Enough workgroups for four per CU, each at least 2048 columns wide; chunks are
  // whole 8-entry groups.
  const int64_t want = (4 * int64_t(device_cu_count()) + rows - 1) / (rows > 0 ? rows : 1);
  const int max_parts = (V + 2047) / 2048;
  n_parts = int(want < 1 ? 1 : (want > max_parts ? max_parts : want));
  chunk = ((V + n_parts - 1) / n_parts + 7) / 8 * 8;
  n_parts = (V + chunk - 1) / chunk;
}

size_t sample_parts_bytes(int64_t rows, int V) {
  int np, ch;
  row_split(rows, V, np, ch);
  return size_t(rows) * size_t(np) * sizeof(RowState);
}

// The passes over the rows alone; n_parts partials a row are left in `part`.
static hipError_t launch_row_pass(const float* logits, int64_t rows, int V, int64_t ld, float inv_t,
                                  bool sample, uint64_t seed, uint64_t stream, RowState* part,
                                  int& np, hipStream_t s) {
  int ch;
  row_split(rows, V, np, ch);
  const dim3 grid(static_cast<unsigned>(rows), static_cast<unsigned>(np));
  if (sample)
    hipLaunchKernelGGL(row_pass_kernel<true>, grid, dim3(kSampleThreads), 0, s, logits, ld, V, np, ch,
                       inv_t, seed, stream, part);
  else
    hipLaunchKernelGGL(row_pass_kernel<false>, grid, dim3(kSampleThreads), 0, s, logits, ld, V, np,
                       ch, inv_t, seed, stream, part);
  return hipGetLastError();
}

hipError_t launch_row_softmax(const float* logits, int64_t rows, int V, int64_t ld, float inv_t,
                              bool sample, uint64_t seed, uint64_t stream, int32_t* tokens,
                              float* lse, void* part_ws, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  int np = 0;
  RowState* part = static_cast<RowState*>(part_ws);
  const hipError_t e = launch_row_pass(logits, rows, V, ld, inv_t, sample, seed, stream, part, np, s);
  if (e != hipSuccess) return e;
  constexpr int kRows = kSampleThreads / 64;
  hipLaunchKernelGGL(row_finish_kernel, dim3(unsigned((rows + kRows - 1) / kRows)),
                     dim3(kSampleThreads), 0, s, part, rows, np, lse, tokens);
  return hipGetLastError();
}

// One workgroup per sequence: its waves finish the log-sum-exps of its K + 1 target rows,
// then the first wave decides: lane i tests slot i (u q < p); n = first rejection or K.
// Writes n, the log-sum-exp of target row n, the verified-token row prefix (drafts 0..n-1)
// and clears the sequence's two draw keys.
constexpr int kDecideThreads = 1024;
constexpr int kMaxSlots = 1025;   // K + 1 target rows

__global__ void __launch_bounds__(kDecideThreads)
accept_decide_kernel(const int32_t* __restrict__ draft, int draft_stride,
                     const float* __restrict__ draft_logits, const float* __restrict__ draft_lse,
                     int64_t ld, const float* __restrict__ target_logits,
                     const RowState* __restrict__ part, int n_parts, int K, int V, float inv_t,
                     uint64_t seed, uint64_t stream, int32_t* __restrict__ n_out,
                     float* __restrict__ lse_out, int32_t* __restrict__ tgt,
                     unsigned long long* __restrict__ keys) {
  __shared__ float lse[kMaxSlots];
  const int s = blockIdx.x;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t t0 = int64_t(s) * (K + 1);
  for (int i = wid; i <= K; i += int(blockDim.x >> 6)) {
    const RowState a = row_combine(part + (t0 + i) * n_parts, n_parts);
    if (lane == 0) lse[i] = a.m + logf(a.s);
  }
  __syncthreads();
  if (wid != 0) return;
  int n = K;
  for (int c0 = 0; c0 < K; c0 += 64) {
    const int i = c0 + lane;
    bool reject = false;
    if (i < K) {
      const int64_t dr = int64_t(s) * draft_stride + i;
      const int x = draft[dr];
      const float q = __expf(draft_logits[dr * ld + x] * inv_t - draft_lse[dr]);
      const float p = __expf(target_logits[(t0 + i) * V + x] * inv_t - lse[i]);
      uint32_t dk[8];
      draws8(seed, stream, uint64_t(s), uint64_t(i >> 3), kPurposeAccept, dk);
      // Below 1 also after rounding, so that a draft with q = p is never rejected.
      const float u = fminf(uniform(dk[i & 7]), 1.f - 5.9604644775390625e-8f);
      reject = !(u * q < p);
    }
    const unsigned long long m = __ballot(reject);
    if (m != 0ull) {
      n = c0 + __ffsll(static_cast<long long>(m)) - 1;
      break;
    }
  }
  for (int i = lane; i <= K; i += 64) tgt[t0 + i] = i < n ? draft[int64_t(s) * draft_stride + i] : -1;
  if (lane == 0) {
    n_out[s] = n;
    lse_out[s] = lse[n];
    keys[2 * s] = 0ull;
    keys[2 * s + 1] = 0ull;
  }
}

// The draw after the decisions, split over the vocabulary: workgroup (s, j) scans
// columns [j*chunk, ...) of row n of sequence s.  Key 0: the race of max(0, p_n - q_n) after
// a rejection, of p_K after K acceptances; key 1: of p_n (used only if the residual has no
// positive entry).  The numerators are probabilities, so the ratios of all workgroups share
// one scale and are the keys' order as they are.  A few thousand columns a sequence and
// workgroup: the launch is one chain of loads, generator rounds and the key reduction (8
// sequences x 129280: 17.2 -> 7.7 us with 16-byte loads ahead of the generator and one key
// reduction in place of two merges of log-sum-exp states).
__global__ void __launch_bounds__(kSampleThreads)
accept_draw_kernel(const float* __restrict__ draft_logits, const float* __restrict__ draft_lse,
                   int64_t ld, int draft_stride, const float* __restrict__ target_logits,
                   const float* __restrict__ target_lse, int K, int V, int chunk, float inv_t,
                   uint64_t seed, uint64_t stream, const int32_t* __restrict__ n_in,
                   unsigned long long* __restrict__ keys) {
  const int s = blockIdx.x, j = blockIdx.y;
  const int n = n_in[s];
  const float* zt = target_logits + (int64_t(s) * (K + 1) + n) * V;
  const float lt = target_lse[s];
  const bool resid = n < K;
  const int64_t dr = int64_t(s) * draft_stride + (resid ? n : 0);
  const float* zd = resid ? draft_logits + dr * ld : zt;   // not read without a rejection
  const float ldr = resid ? draft_lse[dr] : 0.f;
  const bool vec = ((reinterpret_cast<uintptr_t>(zt) | reinterpret_cast<uintptr_t>(zd)) & 15u) == 0;
  const int c0 = j * chunk, c1 = min(V, c0 + chunk);
  unsigned long long ka = 0ull, kb = 0ull;
  for (int g = c0 / 8 + threadIdx.x; 8 * g < c1; g += kSampleThreads) {
    const int v0 = 8 * g, nv = min(8, c1 - v0);
    float t[8], d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (vec && nv == 8) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 a = *reinterpret_cast<const float4*>(zt + v0 + 4 * h);
        t[4 * h] = a.x; t[4 * h + 1] = a.y; t[4 * h + 2] = a.z; t[4 * h + 3] = a.w;
        if (resid) {
          const float4 b = *reinterpret_cast<const float4*>(zd + v0 + 4 * h);
          d[4 * h] = b.x; d[4 * h + 1] = b.y; d[4 * h + 2] = b.z; d[4 * h + 3] = b.w;
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        t[k] = k < nv ? zt[v0 + k] : 0.f;
        if (resid && k < nv) d[k] = zd[v0 + k];
      }
    }
    uint32_t dk[8];
    draws8(seed, stream, uint64_t(s), uint64_t(g), kPurposeResample, dk);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k < nv) {
        const float p = __expf(t[k] * inv_t - lt);
        const float w = resid ? p - __expf(d[k] * inv_t - ldr) : p;
        const unsigned long long key = sample_key(race(w, dk[k]), v0 + k);
        if (w > 0.f && key > ka) ka = key;
        const unsigned long long fall = sample_key(race(p, dk[k]), v0 + k);
        if (resid && p > 0.f && fall > kb) kb = fall;
      }
    }
  }
  __shared__ unsigned long long sh[2][kSampleThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long xa = __shfl_xor(ka, o, kWave), xb = __shfl_xor(kb, o, kWave);
    ka = xa > ka ? xa : ka;
    kb = xb > kb ? xb : kb;
  }
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = ka;
    sh[1][threadIdx.x >> 6] = kb;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long k = 0ull;
    for (int w = 0; w < kSampleThreads / 64; ++w) k = sh[threadIdx.x][w] > k ? sh[threadIdx.x][w] : k;
    if (k != 0ull) atomicMax(keys + 2 * s + threadIdx.x, k);
  }
}

size_t accept_sample_ws_bytes(int n_seq, int K, int V) {
  const size_t rows = size_t(n_seq) * (K + 1);
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  return al(rows * 4) + al(size_t(n_seq) * 4) + al(size_t(n_seq) * 16) + al(rows * 4) +
         al(sample_parts_bytes(int64_t(rows), V));
}

hipError_t launch_accept_sample(const int32_t* draft, int draft_stride, const float* draft_logits,
                                const float* draft_lse, int64_t ld, const float* target_logits,
                                int n_seq, int K, int V, float inv_t, uint64_t seed,
                                uint64_t stream, int32_t* acc, int32_t* anchor, int32_t* offs,
                                int32_t* toks, void* ws, hipStream_t s) {
  const int64_t rows = int64_t(n_seq) * (K + 1);
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  char* p = static_cast<char*>(ws);
  float* tlse = reinterpret_cast<float*>(p);
  p += al(size_t(rows) * 4);
  int32_t* n_buf = reinterpret_cast<int32_t*>(p);
  p += al(size_t(n_seq) * 4);
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(p);
  p += al(size_t(n_seq) * 16);
  int32_t* tgt = reinterpret_cast<int32_t*>(p);
  p += al(size_t(rows) * 4);
  RowState* part = reinterpret_cast<RowState*>(p);
  int tp = 0;
  hipError_t e = launch_row_pass(target_logits, rows, V, V, inv_t, false, 0, 0, part, tp, s);
  if (e != hipSuccess) return e;
  // A wave per target row, up to sixteen.
  const int decide = 64 * (K + 1 < kDecideThreads / 64 ? K + 1 : kDecideThreads / 64);
  hipLaunchKernelGGL(accept_decide_kernel, dim3(n_seq), dim3(decide), 0, s, draft, draft_stride,
                     draft_logits, draft_lse, ld, target_logits, part, tp, K, V, inv_t, seed, stream,
                     n_buf, tlse, tgt, keys);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  int np, ch;
  row_split(n_seq, V, np, ch);
  hipLaunchKernelGGL(accept_draw_kernel, dim3(n_seq, np), dim3(kSampleThreads), 0, s, draft_logits,
                     draft_lse, ld, draft_stride, target_logits, tlse, K, V, ch, inv_t, seed, stream,
                     n_buf, keys);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // The verified tokens of sequence s then read drafts 0..n-1 and the draw, which differs
  // from draft n (a rejected draft has p < q, so its residual weight is 0): greedy
  // acceptance against this row yields n, the draw as next anchor and the commits.
  return launch_accept_drawn(draft, draft_stride, tgt, n_buf, keys, n_seq, K, acc, anchor, offs,
                             toks, s);
}

}  // namespace hdf
