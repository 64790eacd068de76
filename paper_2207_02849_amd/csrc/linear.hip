// Single-layer models (linear and softmax regression with a decay per parameter) that fit one
// compute unit: a whole hypergradient in one workgroup.
//
// With launches for every product such a problem is a chain of dependent launches of 3 to 5 us each, two
// per Neumann step and four per conjugate-gradient step, for a few thousand multiplications.  Here the
// data stay in registers, once by rows and once by columns (a thread holds 32 features of one sample and 32
// samples of one feature), the vectors in LDS, and a step is four workgroup barriers:
//   rows     z = X s           partial sums over 32 features a thread
//   Hessian  R delta = L'' z   a thread per sample
//   columns  X^T R delta       partial sums over 32 samples a thread
//   update   a thread per parameter (s, or q, r, d of conjugate gradient)
// The squared error's Hessian does not depend on the sample: for the Neumann series a launch before forms G = (2 / B)
// X^T X, which takes the data's place in the registers, and a step is one product with it, two barriers, whatever the
// train batch; that launch itself takes 3.5 to 5 ns a sample.  (Conjugate gradient keeps the data: it divides by curvatures that X^T (X d) leaves closer to their true size.)
// The bias is a feature that is 1 for every sample.  All arithmetic in fp32, dot products of conjugate
// gradient in double.
#include "internal.h"

namespace betty {

constexpr int LIN_T = 1024, LIN_CH = 32, LIN_LDS = 152 * 1024;

__host__ __device__ static inline int lin_up(int n) { return (n + LIN_CH - 1) / LIN_CH; }
__host__ __device__ static inline int lin_16(int n) { return (n + 15) & ~15; }

// LDS of a problem in floats: partial sums, the rows' quantities (R delta, softmax probabilities), vectors
static size_t lin_lds_floats(int n, int C, int Bmax, bool cg) {
  return (size_t)C * (LIN_T + 2 * LIN_CH * lin_up(Bmax) + (cg ? 5 : 3) * LIN_CH * lin_up(n));
}

bool linear_fits(int n, int C, int B, int Bv, bool mse, bool cg) {
  if (mse && !cg) B = lin_up(n) * LIN_CH;                // (G in the place of the train batch)
  const int Bm = B > Bv ? B : Bv;
  return n <= LIN_T && Bm <= LIN_T && lin_up(n) * lin_16(Bm) <= LIN_T && lin_up(Bm) * lin_16(n) <= LIN_T &&
         lin_lds_floats(n, C, Bm, cg) * 4 <= LIN_LDS;
}

// X of one side into registers: 32 features of sample t % B, 32 samples of feature t % n (B, n rounded up to 16 lanes)
__device__ __forceinline__ void lin_load(const LinearArgs& a, int side, int n, int t, float (&xr)[LIN_CH], float (&xc)[LIN_CH]) {
  const int B = a.B[side], BR = lin_16(B), NR = lin_16(n);
  const int i = min(t % BR, B - 1), k0 = t / BR * LIN_CH, k = t % NR, r0 = t / NR * LIN_CH;
#pragma unroll
  for (int j = 0; j < LIN_CH; j += 4) {            // (columns beyond n_in and rows beyond B are zero padding)
    const float4 v = k0 < a.n_in ? *(const float4*)(a.X[side] + (long long)i * a.ldx + k0 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    xr[j] = v.x; xr[j + 1] = v.y; xr[j + 2] = v.z; xr[j + 3] = v.w;
  }
#pragma unroll
  for (int j = 0; j < LIN_CH; j += 4) {
    const float4 v = k < a.n_in && r0 < B ? *(const float4*)(a.XT[side] + (long long)k * a.ldxt[side] + r0 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    xc[j] = v.x; xc[j + 1] = v.y; xc[j + 2] = v.z; xc[j + 3] = v.w;
  }
  if (n > a.n_in) {
#pragma unroll
    for (int j = 0; j < LIN_CH; ++j) {
      if (k0 + j == a.n_in) xr[j] = 1.f;
      if (k == a.n_in) xc[j] = r0 + j < B ? 1.f : 0.f;
    }
  }
}

// s += sum_j x[J + j] y(lane j of the same row of 16 lanes).  The broadcast is part of the multiply-add: the
// compiler leaves a move of its own in front of each (1024-sample column sums: twice the instructions).  s_nop: a
// register that a vector instruction has just written may be read across lanes two states later.
template <int J>
__device__ __forceinline__ void lin_fma16(const float (&x)[LIN_CH], float y, float (&s)[4]) {
  asm("s_nop 1\n"
      "v_fmac_f32_dpp %0, %20, %4 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %1, %20, %5 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %2, %20, %6 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %3, %20, %7 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %0, %20, %8 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %1, %20, %9 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %2, %20, %10 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %3, %20, %11 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %0, %20, %12 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %1, %20, %13 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %2, %20, %14 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %3, %20, %15 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %0, %20, %16 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %1, %20, %17 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %2, %20, %18 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %3, %20, %19 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
      : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])
      : "v"(x[J + 0]), "v"(x[J + 1]), "v"(x[J + 2]), "v"(x[J + 3]), "v"(x[J + 4]), "v"(x[J + 5]), "v"(x[J + 6]), "v"(x[J + 7]), "v"(x[J + 8]), "v"(x[J + 9]), "v"(x[J + 10]), "v"(x[J + 11]), "v"(x[J + 12]), "v"(x[J + 13]), "v"(x[J + 14]), "v"(x[J + 15]), "v"(y));
}

// part[c][t] = sum over this thread's 32 entries of x[.] vec[c][first + .]; `first` is the same for 16 lanes, which
// hold one entry each (two reads of LDS; eight of 16 bytes take 8 cycles each)
__device__ __forceinline__ void lin_dot(const float (&x)[LIN_CH], const float* vec, int ld, int first, int C, int t, float* part) {
  const float* v = vec + first + (t & 15);
  int c = 0;
  for (; c + 2 <= C; c += 2) {                     // two classes at once hide each other's latency
    const float y0 = v[c * ld], y1 = v[c * ld + 16], u0 = v[(c + 1) * ld], u1 = v[(c + 1) * ld + 16];
    float s[4] = {0.f, 0.f, 0.f, 0.f}, r[4] = {0.f, 0.f, 0.f, 0.f};
    lin_fma16<0>(x, y0, s);
    lin_fma16<0>(x, u0, r);
    lin_fma16<16>(x, y1, s);
    lin_fma16<16>(x, u1, r);
    part[c * LIN_T + t] = (s[0] + s[1]) + (s[2] + s[3]);
    part[(c + 1) * LIN_T + t] = (r[0] + r[1]) + (r[2] + r[3]);
  }
  if (c < C) {
    const float y0 = v[c * ld], y1 = v[c * ld + 16];
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    lin_fma16<0>(x, y0, s);
    lin_fma16<16>(x, y1, s);
    part[c * LIN_T + t] = (s[0] + s[1]) + (s[2] + s[3]);
  }
}

// sum of m partial sums `pitch` apart, four in flight
__device__ __forceinline__ float lin_total(const float* p, int m, int pitch) {
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  int q = 0;
  for (; q + 4 <= m; q += 4)
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] += p[(q + j) * pitch];
  for (; q < m; ++q) s[0] += p[q * pitch];
  return (s[0] + s[1]) + (s[2] + s[3]);
}

__device__ __forceinline__ double lin_block_sum(double x, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < LIN_T / 64; ++k) s += red[k];
  return s;
}

// 16 wavefronts leave a lane 128 registers: 64 for the data.
template <bool CG, bool GRAM>
__global__ __launch_bounds__(LIN_T) void linear_hypergrad_kernel(LinearArgs a) {
  extern __shared__ float4 lin_smem[];
  __shared__ double red[LIN_T / 64];
  const int t = threadIdx.x, C = a.C, n = a.n_in + a.bias, Q = lin_up(n), NP = Q * LIN_CH, NR = lin_16(n);
  const int BP = lin_up(max(GRAM ? NP : a.B[0], a.B[1])) * LIN_CH;
  float* const part = (float*)lin_smem;            // [C][1024]
  float* const rd = part + C * LIN_T;              // [C][BP]
  float* const pr = rd + C * BP;                   // [C][BP]
  float* const sv = pr + C * BP;                   // [C][NP]: w, then s (Neumann) or d
  float* const gv = sv + C * NP;                   // g, or r
  float* const el = gv + C * NP;                   // 2 exp(lambda)
  float* const qv = el + C * NP;                   // conjugate gradient: q, H d
  float* const hv = qv + C * NP;
  const bool ce = a.loss == BETTY_LOSS_SOFTMAX_CE;

  float xr[LIN_CH], xc[LIN_CH];
  lin_load(a, 1, n, t, xr, xc);
  for (int x = t; x < 2 * C * BP; x += LIN_T) rd[x] = 0.f;
  for (int x = t; x < C * NP; x += LIN_T) {
    const int c = x / NP, k = x % NP;
    sv[x] = k < n ? a.w[k * C + c] : 0.f;
    el[x] = k < n ? 2.f * expf(a.lam[k * C + c]) : 0.f;
  }
  __syncthreads();

  // f(class, feature, position in a vector) for this thread's parameters
  const int c_first = t / n, k_first = t % n, c_next = LIN_T / n, k_next = LIN_T % n;
  auto params = [&](auto f) {
    for (int c = c_first, k = k_first; c < C;) {
      f(c, k, c * NP + k);
      c += c_next; k += k_next;
      if (k >= n) { k -= n; ++c; }
    }
  };
  auto rows = [&](int side) {                      // part = rows of X sv
    const int B = a.B[side];
    const int BR = lin_16(B);
    if (t < Q * BR) lin_dot(xr, sv, NP, t / BR * LIN_CH, C, t, part);
    __syncthreads();
  };
  auto logit = [&](int c, int B) { return lin_total(part + c * LIN_T + t, Q, lin_16(B)); };   // z of sample t
  auto columns = [&](int side) {                   // part = columns of X^T rd
    __syncthreads();
    if (t < lin_up(a.B[side]) * NR) lin_dot(xc, rd, BP, t / NR * LIN_CH, C, t, part);
    __syncthreads();
  };
  auto gradient = [&](int c, int k, int side) { return lin_total(part + c * LIN_T + k, lin_up(a.B[side]), NR); };
  // softmax of sample t's logits into dst
  auto softmax = [&](float* dst, int B) {
    float m = -INFINITY, sum = 0.f;
    for (int c = 0; c < C; ++c) { const float z = logit(c, B); dst[c * BP + t] = z; m = fmaxf(m, z); }
    for (int c = 0; c < C; ++c) { const float e = expf(dst[c * BP + t] - m); dst[c * BP + t] = e; sum += e; }
    const float inv = 1.f / sum;
    for (int c = 0; c < C; ++c) dst[c * BP + t] *= inv;
  };

  // ---- g = gradient of the upper cost at w (validation batch)
  rows(1);
  if (t < a.B[1]) {
    const float s = 1.f / (float)a.B[1];
    if (ce) {
      softmax(rd, a.B[1]);
      const int y = min(max(a.labels[1].y[t], 0), C - 1);
      for (int c = 0; c < C; ++c) rd[c * BP + t] = s * (rd[c * BP + t] - (c == y ? 1.f : 0.f));
    } else {
      const float* target = a.labels[1].target + (long long)t * C;
      for (int c = 0; c < C; ++c) rd[c * BP + t] = s * 2.f * (logit(c, a.B[1]) - target[c]);
    }
  }
  columns(1);
  params([&](int c, int k, int o) { gv[o] = gradient(c, k, 1); });

  const int B = a.B[0];
  // Squared errors of up to 64 features: the outputs do not meet in G, so a wavefront takes one through all steps by itself, a feature
  // a lane and G's columns (the rows, as it is symmetric) in its registers: no barrier between the steps (64 - 1, batch 512, K = 20:
  // 19.6 -> 16.5 us a call; with the vector through v_readlane instead of LDS 22.4).  All 16 wavefronts' loads of G had taken 1.5 us beside one
  // output: 7 - 1, K = 1 7.9 us without this form, 9.7, 8.1 with loads where there is an output.  A single step of more than 32 features stays with
  // the form below (32 - 3 with a bias, K = 1: 9.6, 10.0 us).
  const bool own = GRAM && n <= 64 && (n <= LIN_CH || a.K > 1);
  if (own) {
    const int k = t & 63, kc = min(k, NP - 1), wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (wave < C) {                                // (a wavefront without an output would keep the compute unit's L1 busy for nothing)
      int nl = n;
      asm("" : "+v"(nl));                          // (compared a lane: of a comparison of scalars the compiler makes branches that wait for each load)
#pragma unroll
      for (int j = 0; j < LIN_CH; ++j) xr[j] = a.G[min(j, n - 1) * NP + kc];
      if (n > LIN_CH) {
#pragma unroll
        for (int j = 0; j < LIN_CH; ++j) xc[j] = a.G[min(j + LIN_CH, n - 1) * NP + kc];
      }
#pragma unroll
      for (int j = 0; j < LIN_CH; ++j) { xr[j] = j < nl ? xr[j] : 0.f; xc[j] = j + LIN_CH < nl ? xc[j] : 0.f; }
    }
    __syncthreads();
    for (int c = wave; c < C; c += LIN_T / 64) {
      const float g = k < n ? gv[c * NP + k] : 0.f, e = k < n ? el[c * NP + k] : 0.f;
      float* const v = sv + c * NP;
      float sk = g;
      for (int step = 0; step < a.K; ++step) {
        float h[4] = {0.f, 0.f, 0.f, 0.f}, f[4] = {0.f, 0.f, 0.f, 0.f};
        if (k < NP) v[k] = sk;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        const float y0 = v[k & 15], y1 = v[16 + (k & 15)];
        float y2 = 0.f, y3 = 0.f;
        if (n > LIN_CH) { y2 = v[32 + (k & 15)]; y3 = v[48 + (k & 15)]; }
        lin_fma16<0>(xr, y0, h);
        lin_fma16<16>(xr, y1, h);
        if (n > LIN_CH) {
          lin_fma16<0>(xc, y2, f);
          lin_fma16<16>(xc, y3, f);
        }
        const float hs = ((h[0] + h[1]) + (h[2] + h[3])) + ((f[0] + f[1]) + (f[2] + f[3])) + e * sk;
        sk = k < n ? g + (sk - a.alpha * hs) : 0.f;
      }
      if (k < n) sv[c * NP + k] = sk;
    }
    __syncthreads();
  } else if constexpr (GRAM) {
    const int k = min(t % NR, n - 1), k0 = t / NR * LIN_CH;
#pragma unroll
    for (int j = 0; j < LIN_CH; j += 4) {
      const float4 v = k0 < NP ? *(const float4*)(a.G + k * NP + k0 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
      xr[j] = v.x; xr[j + 1] = v.y; xr[j + 2] = v.z; xr[j + 3] = v.w;
    }
    __syncthreads();
  } else {
    // ---- train batch: probabilities at w
    lin_load(a, 0, n, t, xr, xc);
    __syncthreads();
    if (ce) {
      rows(0);
      if (t < B) softmax(pr, B);
      __syncthreads();
    }
    for (int x = t; x < C * BP; x += LIN_T) if (x % BP >= B) rd[x] = 0.f;      // what the other batch left
  }
  if (!own) {
    for (int x = t; x < C * NP; x += LIN_T) { sv[x] = x % NP < n ? gv[x] : 0.f; if (CG) qv[x] = 0.f; }
    __syncthreads();
  }

  const float si = 1.f / (float)B;
  auto product = [&]() {                           // part = partial sums of the data's part of H sv
    if constexpr (GRAM) {
      if (t < Q * NR) lin_dot(xr, sv, NP, t / NR * LIN_CH, C, t, part);
      __syncthreads();
      return;
    }
    rows(0);
    if (t < B) {
      if (ce) {
        float dot = 0.f;
        for (int c = 0; c < C; ++c) { const float z = logit(c, B); rd[c * BP + t] = z; dot = fmaf(pr[c * BP + t], z, dot); }
        for (int c = 0; c < C; ++c) {
          const float p = pr[c * BP + t];
          rd[c * BP + t] = si * (p * rd[c * BP + t] - p * dot);
        }
      } else {
        for (int c = 0; c < C; ++c) rd[c * BP + t] = si * 2.f * logit(c, B);
      }
    }
    columns(0);
  };

  float rs = 0.f;
  if constexpr (CG) {
    double acc = 0.0;
    params([&](int, int, int o) { const double r = gv[o]; acc += r * r; });
    rs = (float)lin_block_sum(acc, red);
  }
  const int m = GRAM ? Q : lin_up(B);               // partial sums a parameter
  for (int step = 0; step < (own ? 0 : a.K); ++step) {
    product();
    if constexpr (!CG) {
      params([&](int c, int k, int o) {
        const float s = sv[o], hs = lin_total(part + c * LIN_T + k, m, NR) + el[o] * s;
        sv[o] = gv[o] + (s - a.alpha * hs);
      });
    } else {
      double acc = 0.0;
      params([&](int c, int k, int o) {
        const float h = lin_total(part + c * LIN_T + k, m, NR) + el[o] * sv[o];
        hv[o] = h;
        acc += (double)h * (double)sv[o];
      });
      const float den = (float)lin_block_sum(acc, red), f = rs != 0.f && den != 0.f ? rs / den : 0.f;
      acc = 0.0;
      params([&](int, int, int o) {
        qv[o] += f * sv[o];
        const float r = gv[o] - f * hv[o];
        gv[o] = r;
        acc += (double)r * (double)r;
      });
      const float rs_new = (float)lin_block_sum(acc, red), beta = rs != 0.f ? rs_new / rs : 0.f;
      params([&](int, int, int o) { sv[o] = gv[o] + beta * sv[o]; });
      rs = rs_new;
    }
    __syncthreads();
  }
  for (int x = t; x < C * n; x += LIN_T) {
    const int c = x % C, k = x / C, o = c * NP + k;
    const float q = CG ? qv[o] : a.alpha * sv[o];
    a.out[x] = -el[o] * a.w[x] * q;
  }
}

// G = (2 / B) X^T X as [n][NP], features and bias: a workgroup per 16-tile, samples split over its wavefronts
// (lane l holds feature l % 16, samples 4 (l / 16) ... + 3 of both operands; partial tiles summed in wavefront order).
__global__ __launch_bounds__(512) void linear_gram_kernel(LinearArgs a) {
  typedef float f32x4v __attribute__((ext_vector_type(4)));
  constexpr int W = 8;
  __shared__ float part[W][16][17];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = a.n_in + a.bias, NP = lin_up(n) * LIN_CH, tiles = NP / 16;
  const int i0 = (int)blockIdx.x / tiles * 16, j0 = (int)blockIdx.x % tiles * 16, B = a.B[0];
  const int i = i0 + (lane & 15), j = j0 + (lane & 15), k0 = 4 * (lane >> 4);
  auto load = [&](int f, int r0) {                 // (samples beyond B are zero padding)
    if (f < a.n_in) return *(const f32x4v*)(a.XT[0] + (long long)f * a.ldxt[0] + r0);
    f32x4v v = {0.f, 0.f, 0.f, 0.f};
    if (f < n)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = r0 + r < B ? 1.f : 0.f;
    return v;
  };
  f32x4v acc = {0.f, 0.f, 0.f, 0.f};
  const int steps = (B + 15) / 16, per = (steps + W - 1) / W, end = min(steps, (wave + 1) * per);
  for (int s = wave * per; s < end; ++s) {
    const f32x4v x = load(i, 16 * s + k0), y = load(j, 16 * s + k0);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r], y[r], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[wave][4 * (lane >> 4) + r][lane & 15] = acc[r];
  __syncthreads();
  if (t >= 256) return;
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < W; ++w) s += part[w][t >> 4][t & 15];
  if (i0 + (t >> 4) < n) a.G[(i0 + (t >> 4)) * NP + j0 + (t & 15)] = (float)(2.0 / B * s);
}

size_t linear_gram_bytes(int n) { return (size_t)n * lin_up(n) * LIN_CH * 4; }

template <bool CG, bool GRAM>
static void launch_linear(Ctx& ctx, const LinearArgs& a) {
  const int n = a.n_in + a.bias, B = GRAM ? lin_up(n) * LIN_CH : a.B[0];
  const size_t lds = lin_lds_floats(n, a.C, B > a.B[1] ? B : a.B[1], CG) * 4;
  static PerDevice allowed;
  const hipError_t e = allow_lds(allowed, (const void*)linear_hypergrad_kernel<CG, GRAM>, LIN_LDS);
  if (e != hipSuccess) { if (ctx.first_error == hipSuccess) ctx.first_error = e; return; }
  if (GRAM && a.K > 0) {
    const int tiles = lin_up(n) * LIN_CH / 16;
    Launch l(ctx, BETTY_K_GEMM, 2.0 * a.B[0] * n * n);
    linear_gram_kernel<<<tiles * tiles, 512, 0, ctx.stream>>>(a);
  }
  Launch l(ctx, BETTY_K_OTHER, 4.0 * a.K * a.B[0] * n * a.C);
  linear_hypergrad_kernel<CG, GRAM><<<1, LIN_T, lds, ctx.stream>>>(a);
}

void launch_linear_hypergrad(Ctx& ctx, const LinearArgs& a, bool cg) {
  if (cg) launch_linear<true, false>(ctx, a);
  else if (a.G) launch_linear<false, true>(ctx, a);
  else launch_linear<false, false>(ctx, a);
}

}  // namespace betty
