// Tensors that fit one compute unit's LDS (arxiv 2202.09512, Alg. 3 / Eq. 2 for the small end of the paper's
// synthetic sweep): one workgroup per ensemble member keeps its perturbed tensor X^r (Alg. 4, built once per
// launch), A^r and R^r in LDS and runs ALL the requested iterations in one launch.  At these sizes an iteration
// of the general path is ten kernel launches of a few microseconds each: launch latency, not arithmetic.
//
// Same statements as the general path (the n-sized products re-associated the same way), each batched over the
// slices (the R updates of different slices are independent once G is known), so that an iteration costs six
// barriers:
//   G = A^T A;  P_t = X_t A, Q_t = X_t^T A;  S_t = A^T P_t;  R_t <- R_t (*) S_t (/) (G R_t G + eps);
//   Num = sum_t P_t R_t^T + Q_t R_t;  W = sum_t R_t G R_t^T + R_t^T G R_t;  A <- A (*) Num (/) (A W + eps).
//
// The k x k sums are formed in 64 bits, which costs little here: their roundings are common to all entities, and over
// hundreds of iterations they add up along the factors' common scale.
// What bounds it: LDS reads and their latency on ONE compute unit per member.  So a workgroup has as many waves as a
// compute unit holds, the sums are split over neighbouring lanes (4 for the n-long ones of P and Q, 4 or 16 for those of the
// k x k matrices) and added up by lane permutations, a lane of the products takes a row of X for P and the column of the
// same number for Q, which need the same rows of A, and it takes 4 columns of A in one read: 8 multiply-adds for three
// reads.  Per iteration (64 entities, 4 slices, rank 3): 14.6 -> 4.7 us.
// Neighbouring lanes walk down columns of the n x k and of the k x k arrays.  With rows of 16 or 32 floats those reads meet in
// one or two LDS banks (40 entities, 4 slices, rank 32: 353 us per iteration; 258 with 4 waves and unsplit sums before), so
// the rows are spaced (109 us with 4 lanes per sum).
#include "common.h"
#include "kernels.h"

namespace nnr {

constexpr int kTinyThreads = 1024;
constexpr int kTinyMaxN = 64;

// sums over 4 and over 16 neighbouring lanes, all of which take part (the result is in every one of them)
template <int CTRL>
__device__ __forceinline__ float add_permuted(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float quad_sum(float v) { return add_permuted<0x4E>(add_permuted<0xB1>(v)); }   // lane ^ 1, lane ^ 2
template <int CTRL>
__device__ __forceinline__ double add_permuted(double v) {
  return v + __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false),
                              __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false));
}
template <int LANES>
__device__ __forceinline__ double lane_sum(double v) {
  static_assert(LANES == 4 || LANES == 16, "a quad or a row of lanes");
  v = add_permuted<0x4E>(add_permuted<0xB1>(v));
  return LANES == 4 ? v : add_permuted<0x140>(add_permuted<0x141>(v));   // mirrored 8, mirrored 16
}

// Divisor of indices below 2^20 that is not known at compile time: (e + 1/2) / v is at least 1 / (2 v) away from an integer,
// more than the two roundings move it.
struct SmallDiv {
  int v;
  float inv;
  __device__ explicit SmallDiv(int d) : v(d), inv(1.0f / (float)d) {}
  __device__ int div(int e) const { return (int)(((float)e + 0.5f) * inv); }
};

// CK: columns of A that a lane reads at once.  kc: pitch of the n x k arrays, a multiple of CK (the spare columns are zero and
// stay zero); kr: pitch of the k x k matrices.  LN: lanes that share a sum over the entities.
template <int CK, int LN>
__global__ void __launch_bounds__(kTinyThreads)
    tiny_fit_kernel(const float* __restrict__ X, float* __restrict__ A_int, float* __restrict__ R, Dims d, int kc, int kr,
                    int iters, float eps, uint32_t k0, uint32_t k1, float dscaled, int perturb) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int n = (int)d.n, m = d.m, k = d.k, q = d.q, kp = d.kp, kk = k * k, mn = m * n, mkk = m * kk;
  const int ks = k * kr, tid = threadIdx.x;          // ks: floats of a k x k matrix
  const int r = blockIdx.x;                          // ensemble member
  const int ldx = n + 1;                             // row pitch of a slice: column walks stay conflict-free
  float* Xs = lds;                                   // [m][n][ldx]
  float* As = Xs + ((mn * ldx + 3) & ~3);            // [n][kc]
  float* Num = As + n * kc;                          // [n][kc]
  float* Pa = Num + n * kc;                          // [m][n][kc]: X_t A
  float* Qa = Pa + mn * kc;                          // [m][n][kc]: X_t^T A
  float* Rs = Qa + mn * kc;                          // [m][k][kr]
  float* Sa = Rs + m * ks;                           // [m][k][kr]: A^T X_t A
  float* T1 = Sa + m * ks;                           // [m][k][kr]
  float* T2 = T1 + m * ks;                           // [m][k][kr]
  float* Gs = T2 + m * ks;                           // [k][kr]
  float* Ws = Gs + ks;                               // [k][kr]

  // ---- the member's perturbed tensor (one Philox block per element; this member's 16-bit half of it)
  for (int e = tid; e < mn * n; e += kTinyThreads) {
    const int t = e / (n * n), i = (e / n) % n, j = e % n;
    float v = X[e];
    if (perturb) {
      const uint64_t c = (uint64_t)i * (uint64_t)n + (uint64_t)j;
      const u32x4 w = philox4x32_10((uint32_t)c, (uint32_t)(c >> 32), (uint32_t)t, (uint32_t)(r >> 3), k0, k1);
      v = perturbed(v, w, r & 7, dscaled);
    }
    Xs[(t * n + i) * ldx + j] = v;
  }
  for (int e = tid; e < n * kc; e += kTinyThreads) {
    const int i = e / kc, c = e % kc;
    As[e] = c < k ? A_int[((int64_t)i * q + r) * kp + c] : 0.0f;
    Num[e] = 0.0f;
  }
  for (int e = tid; e < mkk; e += kTinyThreads) Rs[e / k * kr + e % k] = R[(int64_t)r * mkk + e];
  __syncthreads();

  const int part = tid & 3, rtid = kTinyThreads - 1 - tid;   // (short work starts at the last threads)
  const int ln = tid % LN, l16 = tid & 15;
  const SmallDiv by_k(k), by_n(n), by_mn(mn);
  const int j0 = part * ((n + 3) >> 2), j1 = j0 + ((n + 3) >> 2) < n ? j0 + ((n + 3) >> 2) : n;
  // (the quarters are read from different places on: rows of A a quarter of n apart would often share their banks)
  const int jfirst = j0 < j1 ? j0 + part % (j1 - j0) : j0;
  for (int it = 0; it < iters; ++it) {
    // P[(t,i)][c] = sum_j X_t[i][j] A[j][c];  Q[(t,i)][c] = sum_j X_t[j][i] A[j][c]: a quarter of the j per lane
    for (int e = tid >> 2; e < mn * (kc / CK); e += kTinyThreads / 4) {
      const int ch = by_mn.div(e), c0 = ch * CK, ti = e - ch * mn, t = by_n.div(ti);
      const float* xrow = Xs + ti * ldx;
      const float* xcol = Xs + t * n * ldx + (ti - t * n);
      float p[CK], y[CK];
#pragma unroll
      for (int u = 0; u < CK; ++u) p[u] = y[u] = 0.0f;
      int j = jfirst;
#pragma unroll 4
      for (int jj = j0; jj < j1; ++jj) {
        float a[CK];
        if constexpr (CK == 4) {
          const float4 v = *reinterpret_cast<const float4*>(As + j * kc + c0);
          a[0] = v.x; a[1] = v.y; a[2] = v.z; a[3] = v.w;
        } else {
          a[0] = As[j * kc + c0];
        }
        const float xr = xrow[j], xc = xcol[j * ldx];
#pragma unroll
        for (int u = 0; u < CK; ++u) {
          p[u] = fmaf(xr, a[u], p[u]);
          y[u] = fmaf(xc, a[u], y[u]);
        }
        j = j + 1 < j1 ? j + 1 : j0;
      }
#pragma unroll
      for (int u = 0; u < CK; ++u) {
        const float ps = quad_sum(p[u]), ys = quad_sum(y[u]);
        if (part == 0) Pa[ti * kc + c0 + u] = ps;
        if (part == 1) Qa[ti * kc + c0 + u] = ys;
      }
    }
    // G[a][b] = sum_i A[i][a] A[i][b]
    for (int e = rtid / LN; e < kk; e += kTinyThreads / LN) {
      const int a = by_k.div(e), b = e - a * k;
      double s = 0.0;
      for (int i = ln; i < n; i += LN) s = fma((double)As[i * kc + a], (double)As[i * kc + b], s);
      s = lane_sum<LN>(s);
      if (ln == 0) Gs[a * kr + b] = (float)s;
    }
    __syncthreads();
    // S[(t,a)][b] = sum_i A[i][a] P_t[i][b];  T1[(t,a)][b] = sum_c R_t[a][c] G[c][b]
    for (int e = tid / LN; e < mkk; e += kTinyThreads / LN) {
      const int ta = by_k.div(e), b = e - ta * k, t = by_k.div(ta), a = ta - t * k;
      double s = 0.0;
      for (int i = ln; i < n; i += LN) s = fma((double)As[i * kc + a], (double)Pa[(t * n + i) * kc + b], s);
      s = lane_sum<LN>(s);
      if (ln == 0) Sa[ta * kr + b] = (float)s;
    }
    for (int e = rtid; e < mkk; e += kTinyThreads) {
      const int ta = by_k.div(e), b = e - ta * k;
      float s = 0.0f;
      for (int c = 0; c < k; ++c) s = fmaf(Rs[ta * kr + c], Gs[c * kr + b], s);
      T1[ta * kr + b] = s;
    }
    __syncthreads();
    // R_t <- R_t (*) S_t (/) (G R_t G + eps), (G R_t G)[a][b] = sum_c G[a][c] T1_t[c][b]
    for (int e = tid; e < mkk; e += kTinyThreads) {
      const int ta = by_k.div(e), b = e - ta * k, t = by_k.div(ta), a = ta - t * k;
      double s = 0.0;
      for (int c = 0; c < k; ++c) s = fma((double)Gs[a * kr + c], (double)T1[(t * k + c) * kr + b], s);
      Rs[ta * kr + b] = Rs[ta * kr + b] * Sa[ta * kr + b] / ((float)s + eps);
    }
    __syncthreads();
    // with the new R_t: Num[i][c] = sum_{(t,b)} P_t[i][b] R_t[c][b] + Q_t[i][b] R_t[b][c], a quarter of the t per lane;
    // T1_t = G R_t^T, T2_t = G R_t
    for (int e = tid >> 2; e < n * k; e += kTinyThreads / 4) {
      const int i = by_k.div(e), c = e - i * k;
      float s = 0.0f;
      for (int t = part; t < m; t += 4) {
        const float *p = Pa + (t * n + i) * kc, *y = Qa + (t * n + i) * kc, *rt = Rs + t * ks;
        for (int b = 0; b < k; ++b) s = fmaf(y[b], rt[b * kr + c], fmaf(p[b], rt[c * kr + b], s));
      }
      s = quad_sum(s);
      if (part == 0) Num[i * kc + c] = s;
    }
    for (int e = rtid; e < mkk; e += kTinyThreads) {
      const int ta = by_k.div(e), b = e - ta * k, t = by_k.div(ta), a = ta - t * k;
      float s1 = 0.0f, s2 = 0.0f;
      for (int c = 0; c < k; ++c) {
        const float g = Gs[a * kr + c];
        s1 = fmaf(g, Rs[(t * k + b) * kr + c], s1);
        s2 = fmaf(g, Rs[(t * k + c) * kr + b], s2);
      }
      T1[ta * kr + b] = s1;
      T2[ta * kr + b] = s2;
    }
    __syncthreads();
    // W[a][b] = sum_{(t,c)} R_t[a][c] (G R_t^T)[c][b] + R_t[c][a] (G R_t)[c][b]
    for (int e = tid >> 4; e < kk; e += kTinyThreads / 16) {
      const int a = by_k.div(e), b = e - a * k;
      double s = 0.0;
      for (int tc = l16; tc < m * k; tc += 16) {
        const int t = by_k.div(tc), c = tc - t * k;
        s = fma((double)Rs[tc * kr + a], (double)T2[tc * kr + b],
                fma((double)Rs[(t * k + a) * kr + c], (double)T1[tc * kr + b], s));
      }
      s = lane_sum<16>(s);
      if (l16 == 0) Ws[a * kr + b] = (float)s;
    }
    __syncthreads();
    // A (*) Num (/) (A W + eps) takes Num's place, and the two arrays change roles
    for (int e = tid; e < n * k; e += kTinyThreads) {
      const int i = by_k.div(e), c = e - i * k;
      float den = 0.0f;
      for (int b = 0; b < k; ++b) den = fmaf(As[i * kc + b], Ws[b * kr + c], den);
      Num[i * kc + c] = As[i * kc + c] * Num[i * kc + c] / (den + eps);
    }
    __syncthreads();
    float* const old = As;
    As = Num;
    Num = old;
  }
  for (int e = tid; e < n * k; e += kTinyThreads) A_int[((int64_t)(e / k) * q + r) * kp + e % k] = As[e / k * kc + e % k];
  for (int e = tid; e < mkk; e += kTinyThreads) R[(int64_t)r * mkk + e] = Rs[e / k * kr + e % k];
}

// with n x k arrays of pitch kc and k x k matrices of pitch kr
static size_t tiny_fit_lds_bytes(const Dims& d, int kc, int kr) {
  const size_t n = (size_t)d.n, m = d.m, k = d.k;
  return (m * n * (n + 1) + 2 * n * kc + 2 * m * n * kc + 4 * m * k * kr + 2 * k * kr) * sizeof(float);
}

// everything within 150 KB of LDS
bool tiny_fit_applies(const Dims& d) { return d.n <= kTinyMaxN && tiny_fit_lds_bytes(d, d.k, d.k) <= 150 * 1024; }

// Columns padded to four and rows spaced against bank conflicts where that fits the LDS; else not spaced; and many small slices
// at ranks 1 and 2 can exceed it padded to four as well: one column at a time then.
TinyPitch tiny_fit_pitch(const Dims& d) {
  const int four = (int)round_up(d.k, 4), spaced = four % 8 == 0 ? four + 4 : four, odd = d.k | 1;
  for (const TinyPitch p : {TinyPitch{4, spaced, odd}, TinyPitch{4, four, d.k}})
    if (tiny_fit_lds_bytes(d, p.kc, p.kr) + 12 <= 160 * 1024) return p;   // (what follows X starts at 16 bytes)
  return TinyPitch{1, d.k, d.k};
}

template <int CK, int LN>
static hipError_t launch_tiny_fit_t(const float* X, float* A_int, float* R, const Dims& d, const TinyPitch& p, int iters, float eps,
                                    uint64_t seed, float delta, hipStream_t s) {
  const size_t lds = tiny_fit_lds_bytes(d, p.kc, p.kr) + 12;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)tiny_fit_kernel<CK, LN>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  hipLaunchKernelGGL((tiny_fit_kernel<CK, LN>), dim3((unsigned)d.q), dim3(kTinyThreads), lds, s, X, A_int, R, d, p.kc, p.kr, iters, eps,
                     (uint32_t)seed, (uint32_t)(seed >> 32), delta * 0x1p-16f, delta != 0.0f ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_tiny_fit(const float* X, float* A_int, float* R, const Dims& d, int iters, float eps, uint64_t seed,
                           float delta, hipStream_t s) {
  if (!tiny_fit_applies(d)) return hipErrorInvalidValue;
  const TinyPitch p = tiny_fit_pitch(d);
  if (p.columns == 1) return launch_tiny_fit_t<1, 16>(X, A_int, R, d, p, iters, eps, seed, delta, s);
  // few long sums are split over 16 lanes, many short ones over 4 (418 sizes, 4 to 64 entities: this line takes 1.002 of the
  // better one's time in the mean; 4 lanes take up to 1.22 of 16 lanes' on the one side, 16 up to 1.5 of 4 lanes' on the other)
  return (int64_t)d.m * d.k * d.k > 2 * d.n ? launch_tiny_fit_t<4, 4>(X, A_int, R, d, p, iters, eps, seed, delta, s)
                                            : launch_tiny_fit_t<4, 16>(X, A_int, R, d, p, iters, eps, seed, delta, s);
}

}  // namespace nnr
