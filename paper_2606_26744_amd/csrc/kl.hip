// LM-head KL distillation forward (Sec. 2.4): for the first P draft positions of every
// block, KL(softmax(t/T) || softmax(z/T)) between the teacher logits t = LMHead of the
// path-mean target state at position a+k-1 and the draft logits z of slot k, the
// cross entropy of the draft logits against the ground truth, and
//     L_KL = T^2 / P * mean_blocks sum_k KL,   L = L_CE + alpha * L_KL.
// Four launches: the teacher states, their projection (the LM-head GEMM of gemm.hip with
// its logits kept), one split pass over the vocabulary of every row pair and every
// cross-entropy row with online log-sum-exps, and the finish.
#include "common.hpp"
#include "kernels.hpp"

namespace hdf {

constexpr int kKlThreads = 256;

__device__ __forceinline__ float to_f32(bf16_t x) { return bf2f(x); }
__device__ __forceinline__ float to_f32(float x) { return x; }
template <typename T>
__device__ __forceinline__ T from_f32(float x);
template <>
__device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return f2bf(x); }
template <>
__device__ __forceinline__ float from_f32<float>(float x) { return x; }

// Eight consecutive elements as floats.
template <typename T>
__device__ __forceinline__ void load8f(const T* p, bool vec, float v[8]) {
  if (vec) {
#pragma unroll
    for (int h = 0; h < 8 * int(sizeof(T)) / 16; ++h) {
      const u32x4 x = ld16(p + h * (16 / int(sizeof(T))));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 2) {
          v[2 * e] = lo_bf(x[e]);
          v[2 * e + 1] = hi_bf(x[e]);
        } else {
          v[4 * h + e] = __uint_as_float(x[e]);
        }
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = to_f32(p[e]);
  }
}

// Teacher state: mean over the m paths, RMSNorm, * gamma, rounded to T.  One workgroup per
// row and eight columns a thread and group (d % 64 == 0, d <= 8192), every path's loads of
// a row in flight together (16 rows x 4 x 4096: 23 -> 6 us against one column a thread and
// load).  vec: H is 16-byte aligned (the state always is).
constexpr int kPoolThreads = 512;

template <typename T>
__global__ void __launch_bounds__(kPoolThreads)
pool_norm_kernel(const T* __restrict__ H, int m, int d, bool vec, const float* __restrict__ gamma,
                 float eps, T* __restrict__ out) {
  constexpr int G = 8192 / (8 * kPoolThreads);
  __shared__ float sh[kPoolThreads / 64];
  const int64_t r = blockIdx.x;
  const T* h = H + r * int64_t(m) * d;
  float x[G][8];
  float ss = 0.f;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int c = (g * kPoolThreads + threadIdx.x) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[g][e] = 0.f;
    if (c < d) {
#pragma unroll 4
      for (int j = 0; j < m; ++j) {
        float v[8];
        load8f(h + int64_t(j) * d + c, vec, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[g][e] += v[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[g][e] /= float(m);
        ss = fmaf(x[g][e], x[g][e], ss);
      }
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < kPoolThreads / 64; ++w) tot += sh[w];
  const float rs = rsqrtf(tot / float(d) + eps);
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int c = (g * kPoolThreads + threadIdx.x) * 8;
    if (c < d) {
      T o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = from_f32<T>(x[g][e] * rs * (gamma ? gamma[c + e] : 1.f));
      u32x4* dst = reinterpret_cast<u32x4*>(out + r * d + c);
      u32x4 q[sizeof(o) / 16];
      __builtin_memcpy(q, o, sizeof(o));
#pragma unroll
      for (int e = 0; e < int(sizeof(o) / 16); ++e) dst[e] = q[e];
    }
  }
}

// Online state of one part of a (teacher, student) row pair at temperature T:
// teacher log-sum-exp (mt, st), a = sum_v exp(t_v/T - mt) * (t_v - z_v)/T, and the
// student log-sum-exp (mz, sz).
struct KlState {
  float mt, st, a, mz, sz;
};

__device__ __forceinline__ void kl_merge(KlState& x, const KlState& y) {
  if (y.st > 0.f) {
    if (x.st == 0.f) {
      x.mt = y.mt; x.st = y.st; x.a = y.a;
    } else if (y.mt > x.mt) {
      const float f = __expf(x.mt - y.mt);
      x.st = x.st * f + y.st; x.a = x.a * f + y.a; x.mt = y.mt;
    } else {
      const float f = __expf(y.mt - x.mt);
      x.st += y.st * f; x.a += y.a * f;
    }
  }
  if (y.sz > 0.f) {
    if (x.sz == 0.f) {
      x.mz = y.mz; x.sz = y.sz;
    } else if (y.mz > x.mz) {
      x.sz = x.sz * __expf(x.mz - y.mz) + y.sz; x.mz = y.mz;
    } else {
      x.sz += y.sz * __expf(y.mz - x.mz);
    }
  }
}

// A part of a cross-entropy row: log-sum-exp state (m, s) of the draft logits.
struct LseState {
  float m, s;
};
__device__ __forceinline__ void lse_merge(LseState& x, const LseState& y) {
  if (y.s > 0.f) {
    if (x.s == 0.f) {
      x = y;
    } else if (y.m > x.m) {
      x.s = x.s * __expf(x.m - y.m) + y.s; x.m = y.m;
    } else {
      x.s += y.s * __expf(y.m - x.m);
    }
  }
}

// Columns v0 .. v0+7 of a row scaled by f; columns from end on are -inf.
__device__ __forceinline__ void load_cols(const float* __restrict__ row, int v0, int end, bool vec,
                                          float f, float x[8]) {
  if (vec && v0 + 8 <= end) {
    load8f(row + v0, true, x);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= f;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = v0 + e < end ? row[v0 + e] * f : -INFINITY;
  }
}

// Log-sum-exp state of eight more values; w[e] = e^(x_e - m).  Returns what the state's
// earlier sums were scaled by.  While every value was -inf (masked columns), the exponents
// refer to 0, so that the sums stay 0.
__device__ __forceinline__ float lse_add8(float& m, float& s, const float x[8], float w[8]) {
  float mn = m;
#pragma unroll
  for (int e = 0; e < 8; ++e) mn = fmaxf(mn, x[e]);
  const float ref = mn == -INFINITY ? 0.f : mn;
  float add = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    w[e] = __expf(x[e] - ref);
    add += w[e];
  }
  const float down = __expf(m - ref);
  s = s * down + add;
  m = mn;
  return down;
}

// One launch over both kinds of rows (chunks of whole groups of eight columns): the first
// R * kl_parts workgroups take the parts of row pair i = s*P + (k-1) (teacher row i of
// tl [n*P][V]; student row s*B + k of zl), the others those of the cross-entropy rows
// s*B + k, k = 1..B-1.  Bound by the streams of the logits (8 x 15 rows x 129280 and 16
// pairs: 63 + 17 MB in 16 us; two launches, one of them a column a thread and load, 23 us).
__global__ void __launch_bounds__(kKlThreads)
kl_pass_kernel(const float* __restrict__ tl, const float* __restrict__ zl, int64_t ld, int B, int P,
               int V, int64_t pair_wgs, int kl_parts, int kl_chunk, int ce_parts, int ce_chunk,
               float inv_t, KlState* __restrict__ kl_part, LseState* __restrict__ ce_part) {
  __shared__ KlState sh[kKlThreads / 64];
  const bool pair = int64_t(blockIdx.x) < pair_wgs;
  const int64_t b = pair ? blockIdx.x : blockIdx.x - pair_wgs;
  const int parts = pair ? kl_parts : ce_parts, chunk = pair ? kl_chunk : ce_chunk;
  const int64_t i = b / parts;
  const int j = int(b - i * parts);
  const int per = pair ? P : B - 1;
  const int64_t s = i / per, k = i - s * per + 1;
  const float* z = zl + (s * B + k) * ld;
  const bool vz = (reinterpret_cast<uintptr_t>(z) & 15u) == 0;
  const int c0 = j * chunk, c1 = min(V, c0 + chunk);
  KlState st{-INFINITY, 0.f, 0.f, -INFINITY, 0.f};
  if (pair) {
    const float* t = tl + i * int64_t(V);
    const bool vt = (reinterpret_cast<uintptr_t>(t) & 15u) == 0;
    for (int v = c0 + 8 * int(threadIdx.x); v < c1; v += 8 * kKlThreads) {
      float tt[8], zz[8], wt[8], wz[8];
      load_cols(t, v, c1, vt, inv_t, tt);
      load_cols(z, v, c1, vz, inv_t, zz);
      const float down = lse_add8(st.mt, st.st, tt, wt);
      float a = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) a = wt[e] > 0.f ? fmaf(wt[e], tt[e] - zz[e], a) : a;
      st.a = st.a * down + a;
      lse_add8(st.mz, st.sz, zz, wz);
    }
  } else {
    constexpr int Q = 4;   // groups whose loads are in flight together
    for (int v = c0 + 8 * int(threadIdx.x); v < c1; v += 8 * kKlThreads * Q) {
      float zz[Q][8], wz[8];
#pragma unroll
      for (int q = 0; q < Q; ++q) load_cols(z, v + 8 * kKlThreads * q, c1, vz, 1.f, zz[q]);
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (v + 8 * kKlThreads * q < c1) lse_add8(st.mz, st.sz, zz[q], wz);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    KlState y{__shfl_xor(st.mt, o, kWave), __shfl_xor(st.st, o, kWave), __shfl_xor(st.a, o, kWave),
              __shfl_xor(st.mz, o, kWave), __shfl_xor(st.sz, o, kWave)};
    kl_merge(st, y);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = st;
  __syncthreads();
  if (threadIdx.x == 0) {
    KlState x = sh[0];
    for (int w = 1; w < kKlThreads / 64; ++w) kl_merge(x, sh[w]);
    if (pair)
      kl_part[b] = x;
    else
      ce_part[b] = LseState{x.mz, x.sz};
  }
}

// kl[i] = a/st - (mt + log st) + (mz + log sz); ce from the student log-sum-exps; losses.
// One workgroup.  Row pairs of more than eight parts take a wave each (a part a lane; one
// thread walking 64 parts took 33 us), all other rows a thread.
constexpr int kFinishThreads = 1024;

__device__ __forceinline__ float kl_value(const KlState& x) {
  return x.a / x.st - (x.mt + logf(x.st)) + (x.mz + logf(x.sz));
}

__global__ void __launch_bounds__(kFinishThreads)
kl_finish_kernel(const KlState* __restrict__ kl_part, int kl_parts,
                 const LseState* __restrict__ ce_part, int ce_parts, int n_seq, int P, int B,
                 const float* __restrict__ zl, int64_t ld, const int32_t* __restrict__ labels,
                 float T, float alpha, float* __restrict__ kl, float* __restrict__ ce,
                 float* __restrict__ loss) {
  constexpr int W = kFinishThreads / 64;
  __shared__ float sh[2][W];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  float skl = 0.f, sce = 0.f;
  if (kl_parts > 8) {
    for (int i = wid; i < n_seq * P; i += W) {
      KlState x{-INFINITY, 0.f, 0.f, -INFINITY, 0.f};
      for (int j = lane; j < kl_parts; j += 64) kl_merge(x, kl_part[int64_t(i) * kl_parts + j]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        KlState y{__shfl_xor(x.mt, o, kWave), __shfl_xor(x.st, o, kWave), __shfl_xor(x.a, o, kWave),
                  __shfl_xor(x.mz, o, kWave), __shfl_xor(x.sz, o, kWave)};
        kl_merge(x, y);
      }
      if (lane == 0) {
        const float v = kl_value(x);
        kl[i] = v;
        skl += v;
      }
    }
  } else {
    for (int i = threadIdx.x; i < n_seq * P; i += kFinishThreads) {
      KlState x = kl_part[int64_t(i) * kl_parts];
      for (int j = 1; j < kl_parts; ++j) kl_merge(x, kl_part[int64_t(i) * kl_parts + j]);
      const float v = kl_value(x);
      kl[i] = v;
      skl += v;
    }
  }
  const int K = B - 1;
  if (labels != nullptr) {
    for (int i = threadIdx.x; i < n_seq * K; i += kFinishThreads) {
      const int64_t s = i / K, k = i - s * K + 1;
      const float at = zl[(s * B + k) * ld + labels[i]];
      LseState x = ce_part[int64_t(i) * ce_parts];
#pragma unroll 8
      for (int j = 1; j < ce_parts; ++j) lse_merge(x, ce_part[int64_t(i) * ce_parts + j]);
      const float v = x.m + logf(x.s) - at;
      if (ce != nullptr) ce[i] = v;
      sce += v;
    }
  }
  skl = wave_sum(skl);
  sce = wave_sum(sce);
  if (lane == 0) {
    sh[0][wid] = skl;
    sh[1][wid] = sce;
  }
  __syncthreads();
  if (threadIdx.x == 0 && loss != nullptr) {
    float a = 0.f, c = 0.f;
    for (int w = 0; w < W; ++w) {
      a += sh[0][w];
      c += sh[1][w];
    }
    const float l_kl = T * T / float(P) * a / float(n_seq);
    const float l_ce = labels != nullptr ? c / float(n_seq * K) : 0.f;
    loss[0] = l_kl;
    loss[1] = l_ce;
    loss[2] = l_ce + alpha * l_kl;
  }
}

// Parts of a row of V columns and the columns of each (whole groups of eight): four
// workgroups per CU over all rows, at least 2048 columns each.
static int row_parts(int64_t rows, int V, int& chunk) {
  const int64_t want = (4 * int64_t(device_cu_count()) + rows - 1) / (rows > 0 ? rows : 1);
  const int max_parts = (V + 2047) / 2048;
  const int np = int(want < 1 ? 1 : (want > max_parts ? max_parts : want));
  chunk = ((V + np - 1) / np + 7) / 8 * 8;
  return (V + chunk - 1) / chunk;
}

static size_t al256(size_t x) { return (x + 255) / 256 * 256; }

size_t kl_ws_bytes(int n_seq, int B, int P, int d, int V, bool bf16) {
  const size_t R = size_t(n_seq) * P, C = size_t(n_seq) * (B - 1);
  int ch;
  const size_t np = size_t(row_parts(int64_t(R), V, ch)), nc = size_t(row_parts(int64_t(C), V, ch));
  return al256(R * d * (bf16 ? 2 : 4)) + al256(R * 8) + al256(R * size_t(V) * 4) +
         al256(R * np * sizeof(KlState)) + al256(C * nc * sizeof(LseState));
}

hipError_t launch_kl_forward(bool bf16, const void* H_pos, int m, const float* gamma, float eps,
                             const void* W_lm, int d, int V, const float* zl, int64_t ld, int B,
                             const int32_t* labels, int n_seq, int P, float T, float alpha,
                             float* kl, float* ce, float* loss, void* ws, hipStream_t s) {
  const int64_t R = int64_t(n_seq) * P, C = int64_t(n_seq) * (B - 1);
  char* p = static_cast<char*>(ws);
  void* th = p;                       p += al256(size_t(R) * d * (bf16 ? 2 : 4));
  auto* keys = reinterpret_cast<unsigned long long*>(p); p += al256(size_t(R) * 8);
  auto* tl = reinterpret_cast<float*>(p);               p += al256(size_t(R) * V * 4);
  int kch, cch;
  const int np = row_parts(R, V, kch), nc = row_parts(C, V, cch);
  auto* part = reinterpret_cast<KlState*>(p);           p += al256(size_t(R) * np * sizeof(KlState));
  auto* cpart = reinterpret_cast<LseState*>(p);
  const bool vec = (reinterpret_cast<uintptr_t>(H_pos) & 15u) == 0;
  if (bf16)
    hipLaunchKernelGGL(pool_norm_kernel<bf16_t>, dim3(unsigned(R)), dim3(kPoolThreads), 0, s,
                       static_cast<const bf16_t*>(H_pos), m, d, vec, gamma, eps,
                       static_cast<bf16_t*>(th));
  else
    hipLaunchKernelGGL(pool_norm_kernel<float>, dim3(unsigned(R)), dim3(kPoolThreads), 0, s,
                       static_cast<const float*>(H_pos), m, d, vec, gamma, eps,
                       static_cast<float*>(th));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Only the logits are used: the argmax keys stay unread, whatever they held before.
  e = launch_lm_head_keys(bf16, th, W_lm, R, d, V, keys, tl, s);
  if (e != hipSuccess) return e;
  const int64_t pair_wgs = R * np, wgs = pair_wgs + (labels != nullptr ? C * nc : 0);
  hipLaunchKernelGGL(kl_pass_kernel, dim3(unsigned(wgs)), dim3(kKlThreads), 0, s, tl, zl, ld, B, P,
                     V, pair_wgs, np, kch, nc, cch, 1.f / T, part, cpart);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kl_finish_kernel, dim3(1), dim3(kFinishThreads), 0, s, part, np, cpart, nc,
                     n_seq, P, B, zl, ld, labels, T, alpha, kl, ce, loss);
  return hipGetLastError();
}

}  // namespace hdf
