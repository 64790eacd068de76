// Non-GEMM kernels of the hypergradient path: conversion of flat fp32 parameters into GEMM
// operands in both orientations, the row-wise loss kernels, the two narrow-output-layer kernels
// (last layer of the first-order and of the R-op passes when the output has at most 16 columns),
// the weight-net kernels, and the streaming kernels over the flat parameter-shaped vectors
// (finite-difference steps, conjugate gradient, mixed VJPs, Adam).
#include <algorithm>

#include "internal.h"

namespace betty {

// ------------------------------------------------------------------------------------------
// small device helpers
// ------------------------------------------------------------------------------------------

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

// sum over a 256-thread block, result valid in every thread; fixed combination order
template <typename R>
__device__ __forceinline__ R block_sum(R x, R* smem4) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) smem4[threadIdx.x >> 6] = x;
  __syncthreads();
  return smem4[0] + smem4[1] + smem4[2] + smem4[3];
}

template <typename T> __device__ __forceinline__ T from_float(float x);
template <> __device__ __forceinline__ float from_float<float>(float x) { return x; }
template <> __device__ __forceinline__ __bf16 from_float<__bf16>(float x) { return (__bf16)x; }  // RNE
template <typename T> __device__ __forceinline__ float to_float(T x) { return (float)x; }

// ------------------------------------------------------------------------------------------
// operand conversion: fp32 source -> operand type, row-major and transposed, through a 64x64
// LDS tile; up to MAX_CONVERTS matrices per launch
// ------------------------------------------------------------------------------------------

// four consecutive elements of the operand type as one store
template <typename T> __device__ __forceinline__ void store_quad(T* p, float a, float b, float c, float d);
template <> __device__ __forceinline__ void store_quad<float>(float* p, float a, float b, float c, float d) {
  *(float4*)p = make_float4(a, b, c, d);
}
template <> __device__ __forceinline__ void store_quad<__bf16>(__bf16* p, float a, float b, float c, float d) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
  bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
  *(bf16x4*)p = v;
}

// Bound by latency for the small layers and by memory for the large ones: every load of a tile is
// requested before the first is used (positions are clamped into the matrix instead of being
// predicated; a load inside control flow is waited for before the next one starts).  A 784 x 10 matrix:
// 8 us with predicated loads, 3.6 us; 5.3M parameters: 13.6 us = 4.6 TB/s either way.
template <typename T, int N, int NT>
__global__ __launch_bounds__(NT) void convert_batch_kernel(ConvertBatchT<N> b) {
  constexpr int Q = 1024 / NT, QS = NT / 16, E = 4096 / NT, ES = NT / 64;      // quads, elements a thread; their distance in rows
  __shared__ float tile[64][65];
  int bid = blockIdx.x, ji = 0;
  while (ji + 1 < b.n && bid >= b.block_begin[ji + 1]) ++ji;
  const ConvertJob& j = b.j[ji];
  if (b.table && bid == 0 && threadIdx.x < 2) b.table[threadIdx.x] = b.labels[threadIdx.x];
  bid -= b.block_begin[ji];
  const int tiles_x = (j.cols + 63) / 64;
  const int c0 = (bid % tiles_x) * 64, r0 = (bid / tiles_x) * 64;
  T* out = (T*)j.out;
  T* outT = (T*)j.outT;
  // Four elements per thread and access when the source rows and all destinations allow aligned
  // 16-byte loads (every weight matrix whose width is a multiple of four); else one by one.
  const bool quads = j.cols % 4 == 0 && j.lds % 4 == 0 && j.ld % 4 == 0 && j.ldT % 4 == 0 &&
                     ((uintptr_t)j.src & 15) == 0 && ((uintptr_t)j.out & 15) == 0 && ((uintptr_t)j.outT & 15) == 0 &&
                     ((uintptr_t)j.out32 & 15) == 0 && ((uintptr_t)j.outT32 & 15) == 0;
  if (quads) {
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int c = c0 + 4 * tx;
    float4 v[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i)
      v[i] = *(const float4*)(j.src + (long long)min(r0 + ty + QS * i, j.rows - 1) * j.lds + min(c, j.cols - 4));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int rl = ty + QS * i, r = r0 + rl;
      if (r < j.rows && c < j.cols) {
        if (out) store_quad<T>(out + (long long)r * j.ld + c, v[i].x, v[i].y, v[i].z, v[i].w);
        if (j.out32) store_quad<float>(j.out32 + (long long)r * j.ld + c, v[i].x, v[i].y, v[i].z, v[i].w);
      }
      tile[rl][4 * tx] = v[i].x; tile[rl][4 * tx + 1] = v[i].y; tile[rl][4 * tx + 2] = v[i].z; tile[rl][4 * tx + 3] = v[i].w;
    }
    if (!outT && !j.outT32) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int cl = ty + QS * i, cc = c0 + cl, r = r0 + 4 * tx;
      if (cc >= j.cols || r >= j.rows) continue;
      const float v0 = tile[4 * tx][cl], v1 = tile[4 * tx + 1][cl], v2 = tile[4 * tx + 2][cl], v3 = tile[4 * tx + 3][cl];
      T* o = outT ? outT + (long long)cc * j.ldT + r : nullptr;
      float* o32 = j.outT32 ? j.outT32 + (long long)cc * j.ldT + r : nullptr;
      if (r + 3 < j.rows) {
        if (o) store_quad<T>(o, v0, v1, v2, v3);
        if (o32) store_quad<float>(o32, v0, v1, v2, v3);
      } else {                                     // last rows of a height that is no multiple of four
        const float w[4] = {v0, v1, v2, v3};
        for (int k = 0; k < 4 && r + k < j.rows; ++k) {
          if (o) o[k] = from_float<T>(w[k]);
          if (o32) o32[k] = w[k];
        }
      }
    }
    return;
  }
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  float v[E];
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = j.src[(long long)min(r0 + ty + ES * i, j.rows - 1) * j.lds + min(c0 + tx, j.cols - 1)];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int r = r0 + ty + ES * i, c = c0 + tx;
    if (r < j.rows && c < j.cols) {
      if (out) out[(long long)r * j.ld + c] = from_float<T>(v[i]);
      if (j.out32) j.out32[(long long)r * j.ld + c] = v[i];
    }
    tile[ty + ES * i][tx] = v[i];
  }
  if (!outT && !j.outT32) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int c = c0 + ty + ES * i, r = r0 + tx;
    if (r < j.rows && c < j.cols) {
      if (outT) outT[(long long)c * j.ldT + r] = from_float<T>(tile[tx][ty + ES * i]);
      if (j.outT32) j.outT32[(long long)c * j.ldT + r] = tile[tx][ty + ES * i];
    }
  }
}

// 1024 threads a tile while a compute unit has four tiles at most: a thread's address arithmetic and stores, one after the other, are what
// such a launch waits for (steps of 1023-509-251-10, three conversions: 135.1 -> 130.1 us; product of 777-301-65-33 60.6 -> 59.5);
// beyond, 256, whose four loads a thread keep more bytes in flight.
constexpr int CONVERT_WIDE = 1024;
template <typename T, int N>
static void launch_convert(Ctx& ctx, bool wide, int blocks, const ConvertBatchT<N>& b) {
  if (wide) convert_batch_kernel<T, N, 1024><<<blocks, 1024, 0, ctx.stream>>>(b);
  else convert_batch_kernel<T, N, 256><<<blocks, 256, 0, ctx.stream>>>(b);
}

void launch_convert_batch(Ctx& ctx, Elem elem, ConvertBatch& b) {
  int blocks = 0;
  double bytes = 0;
  for (int i = 0; i < b.n; ++i) {
    const ConvertJob& j = b.j[i];
    b.block_begin[i] = blocks;
    blocks += ((j.cols + 63) / 64) * ((j.rows + 63) / 64);
    bytes += (double)j.rows * j.cols * (4.0 + ((j.out ? 1 : 0) + (j.outT ? 1 : 0)) * elem_size(elem) +
                                        ((j.out32 ? 1 : 0) + (j.outT32 ? 1 : 0)) * 4.0);
  }
  b.block_begin[b.n] = blocks;
  if (blocks <= 0) return;
  Launch l(ctx, BETTY_K_SHADOW, 0, bytes);
  const bool wide = blocks <= CONVERT_WIDE;
  if (b.n > FEW_CONVERTS) {
    if (elem == ELEM_BF16) launch_convert<__bf16>(ctx, wide, blocks, b);
    else launch_convert<float>(ctx, wide, blocks, b);
    return;
  }
  ConvertBatchT<FEW_CONVERTS> few;
  few.n = b.n; few.table = b.table;
  for (int i = 0; i <= b.n; ++i) few.block_begin[i] = b.block_begin[i];
  for (int i = 0; i < b.n; ++i) few.j[i] = b.j[i];
  for (int i = 0; i < 2; ++i) few.labels[i] = b.labels[i];
  if (elem == ELEM_BF16) launch_convert<__bf16>(ctx, wide, blocks, few);
  else launch_convert<float>(ctx, wide, blocks, few);
}

// (a workgroup's 2048 elements are a whole number of 64-element groups, so the result may take the place of the
// sums: everything is read before the barrier)
template <typename T>
__global__ __launch_bounds__(256) void accumulate_kernel(AccumulateBatch b) {
  int bid = blockIdx.x, ji = 0;
  while (ji + 1 < b.n && bid >= b.block_begin[ji + 1]) ++ji;
  const AccumulateJob& j = b.j[ji];
  const size_t i = ((size_t)(bid - b.block_begin[ji]) * 256 + threadIdx.x) * 8;   // < j.n, a multiple of 2048
  typedef __attribute__((__vector_size__(8 * sizeof(T)))) T vecT;
  vecT r = *(const vecT*)((const T*)j.r + i);
  float s[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) s[k] = (b.first ? 0.f : j.beta * j.sum[i + k]) + (float)r[k];
  if (!b.last) {
    *(float4*)(j.sum + i) = make_float4(s[0], s[1], s[2], s[3]);
    *(float4*)(j.sum + i + 4) = make_float4(s[4], s[5], s[6], s[7]);
  } else if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = s[k];
    *(vecT*)((T*)j.r + i) = r;
  } else {
    vecT rem;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      r[k] = (T)s[k];
      rem[k] = (T)(s[k] - (float)r[k]);
    }
    __syncthreads();
    T* o = (T*)j.sum + 2 * (i & ~(size_t)63) + (i & 63);
    *(vecT*)o = r;
    *(vecT*)(o + 64) = rem;
  }
}

void launch_accumulate(Ctx& ctx, Elem elem, AccumulateBatch& b) {
  int blocks = 0;
  double bytes = 0;
  for (int i = 0; i < b.n; ++i) {
    b.block_begin[i] = blocks;
    blocks += (int)(b.j[i].n / 2048);
    bytes += (double)b.j[i].n * (8.0 + elem_size(elem));
  }
  b.block_begin[b.n] = blocks;
  if (blocks <= 0) return;
  Launch l(ctx, BETTY_K_VECTOR, 0, bytes);
  if (elem == ELEM_BF16) accumulate_kernel<__bf16><<<blocks, 256, 0, ctx.stream>>>(b);
  else accumulate_kernel<float><<<blocks, 256, 0, ctx.stream>>>(b);
}

// ------------------------------------------------------------------------------------------
// row-wise loss kernels: one wavefront per sample
// ------------------------------------------------------------------------------------------
//
// A workgroup owns ROWS samples and COLS of the C columns (16 and 256; 4 and 64 for models of up to 64 outputs,
// whose launches are bound by latency): each wavefront keeps its row in registers (up to 64 REGS columns), forms the
// row's sums over all of it (again in every slice of columns: a few KB from L2), writes its slice, and leaves it in LDS,
// from where the transposed copy goes out four samples a store.  With one wavefront per sample on its own, a store of
// the transposed copy touched 64 lines for 2 bytes each and every pass over the row waited for
// memory: 512 x 1000 in bf16 17.3 us, now 7.8, the Hessian's rows 15.3 us, now 5.8; 100 x 10 3.9 us either way (4.9 with 16
// samples a workgroup).
constexpr int lr_rows(int regs) { return regs == 1 ? 4 : 16; }
constexpr int lr_cols(int regs) { return regs == 1 ? 64 : 256; }
static int lr_regs(int C) { return C <= 64 ? 1 : C <= 256 ? 4 : 16; }
__host__ __device__ constexpr int lr_up(int n, int m) { return (n + m - 1) / m; }

// f(k, c) for the columns c = lane + 64 k of a row that are kept in registers, g(c) for those beyond
template <int REGS, typename F, typename G>
__device__ __forceinline__ void row_columns(int lane, int C, F f, G g) {
#pragma unroll
  for (int k = 0; k < REGS; ++k)
    if (lane + 64 * k < C) f(k, lane + 64 * k);
  if constexpr (REGS == 16)
    for (int c = lane + 64 * REGS; c < C; c += 64) g(c);
}

// transposed copy of the tile [column][row] (rows beyond the batch hold zeros: padding of the operand)
template <int ROWS, int COLS, typename T>
__device__ __forceinline__ void store_rows_transposed(const T (*tile)[ROWS + 4], T* Dt, int ldDt, int i0, int c0, int C) {
  __syncthreads();
  constexpr int Q = ROWS / 4;                      // stores a column
  const int t = threadIdx.x, c = c0 + t / Q, q = 4 * (t % Q);
  typedef __attribute__((__vector_size__(4 * sizeof(T)))) T quad;
  if (t < COLS * Q && c < C) *(quad*)(Dt + (long long)c * ldDt + i0 + q) = *(const quad*)&tile[t / Q][q];
}

template <typename T, int REGS>
__global__ __launch_bounds__(64 * lr_rows(REGS)) void loss_rows_kernel(LossBatch lb) {
  constexpr int ROWS = lr_rows(REGS), COLS = lr_cols(REGS);
  __shared__ __attribute__((aligned(16))) T tile[COLS][ROWS + 4];
  const int slices = lr_up(lb.a[0].C, COLS), blocks0 = lr_up(lb.a[0].rows, ROWS) * slices;
  const int which = (lb.n > 1 && (int)blockIdx.x >= blocks0) ? 1 : 0;
  const LossArgs& a = lb.a[which];
  const int bid = (int)blockIdx.x - (which ? blocks0 : 0), slice = bid % slices, c0 = slice * COLS;
  const int i0 = bid / slices * ROWS, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, C = a.C;
  const bool live = i0 + wave < a.rows;
  const int row = live ? i0 + wave : a.rows - 1;
  const float* z = a.Z + (long long)row * a.ldz;
  const Labels lab = *a.labels;
  const bool ce = a.loss == BETTY_LOSS_SOFTMAX_CE;
  const float* t = ce ? nullptr : lab.target + (long long)row * C;
  float zr[REGS], ell, m = 0.f, sum = 1.f;
  int y = 0;
#pragma unroll
  for (int k = 0; k < REGS; ++k) zr[k] = lane + 64 * k < C ? z[lane + 64 * k] : 0.f;
  if (ce) {
    // a label outside [0, C) is clamped into the range, for the gather and the one-hot alike
    y = min(max(lab.y[row], 0), C - 1);
    const float zy = z[y];                         // integer gather of the label's logit
    m = -INFINITY;
    row_columns<REGS>(lane, C, [&](int k, int) { m = fmaxf(m, zr[k]); }, [&](int c) { m = fmaxf(m, z[c]); });
    m = wave_max(m);
    sum = 0.f;
    row_columns<REGS>(lane, C, [&](int k, int) { sum += expf(zr[k] - m); }, [&](int c) { sum += expf(z[c] - m); });
    sum = wave_sum(sum);
    ell = logf(sum) + m - zy;
  } else {
    float acc = 0.f;
    row_columns<REGS>(lane, C, [&](int k, int c) { const float r = zr[k] - t[c]; acc += r * r; },
                [&](int c) { const float r = z[c] - t[c]; acc += r * r; });
    ell = wave_sum(acc);
  }
  float omega = 1.f;
  const bool first = live && slice == 0 && lane == 0;
  if (a.reweight && a.omega_fixed) {
    omega = a.omega_fixed[row];
  } else if (a.reweight) {
    const int H = a.hidden;
    float part = 0.f;
    for (int j = lane; j < H; j += 64)
      part += a.theta[2 * H + j] * fmaxf(a.theta[j] * ell + a.theta[H + j], 0.f);
    part = wave_sum(part) + a.theta[3 * H];
    omega = 1.f / (1.f + expf(-part));
    // sigmoid'(x) = sigmoid(x) sigmoid(-x): no 1 - omega, which loses every digit once omega rounds to 1
    if (first && a.dsig) a.dsig[row] = omega / (1.f + expf(part));
  }
  const float s = omega * a.inv_batch;
  if (first) { a.ell[row] = ell; a.s[row] = s; a.omega[row] = omega; }
  T* D = (T*)a.D + (long long)row * a.ldD;
  float* P = a.P + (long long)row * a.ldz;
  const float inv = 1.f / sum;
#pragma unroll
  for (int k = 0; k < COLS / 64; ++k) {
    const int c = c0 + lane + 64 * k;
    T dv = from_float<T>(0.f);
    if (live && c < C) {
      const float zc = z[c];
      if (ce) {
        const float p = expf(zc - m) * inv;
        P[c] = p;
        dv = from_float<T>(s * (p - (c == y ? 1.f : 0.f)));
      } else {
        dv = from_float<T>(s * 2.f * (zc - t[c]));
      }
      D[c] = dv;
    }
    tile[lane + 64 * k][wave] = dv;
  }
  store_rows_transposed<ROWS, COLS, T>(tile, (T*)a.Dt, a.ldDt, i0, c0, C);
}

template <int REGS>
static void launch_loss_rows_of(hipStream_t st, Elem elem, const LossBatch& lb) {
  int blocks = 0;
  for (int i = 0; i < lb.n; ++i) blocks += lr_up(lb.a[i].rows, lr_rows(REGS)) * lr_up(lb.a[0].C, lr_cols(REGS));
  if (blocks <= 0) return;
  if (elem == ELEM_BF16) loss_rows_kernel<__bf16, REGS><<<blocks, 64 * lr_rows(REGS), 0, st>>>(lb);
  else loss_rows_kernel<float, REGS><<<blocks, 64 * lr_rows(REGS), 0, st>>>(lb);
}
void launch_loss_rows(Ctx& ctx, Elem elem, const LossBatch& lb) {
  if (lb.n <= 0) return;
  Launch l(ctx, BETTY_K_LOSS);
  const int regs = lr_regs(lb.a[0].C);
  if (regs == 1) launch_loss_rows_of<1>(ctx.stream, elem, lb);
  else if (regs == 4) launch_loss_rows_of<4>(ctx.stream, elem, lb);
  else launch_loss_rows_of<16>(ctx.stream, elem, lb);
}

template <typename T, int REGS>
__global__ __launch_bounds__(64 * lr_rows(REGS)) void loss_hessian_rows_kernel(int loss, const float* P, const float* Rz,
                                                                               long long ld, const float* s, int rows,
                                                                               int C, T* D, int ldD, T* Dt, int ldDt) {
  constexpr int ROWS = lr_rows(REGS), COLS = lr_cols(REGS);
  __shared__ __attribute__((aligned(16))) T tile[COLS][ROWS + 4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c0 = blockIdx.y * COLS, i0 = blockIdx.x * ROWS;
  const bool live = i0 + wave < rows, ce = loss == BETTY_LOSS_SOFTMAX_CE;
  const int row = live ? i0 + wave : rows - 1;
  const float* rz = Rz + (long long)row * ld;
  const float* p = P + (long long)row * ld;
  const float si = s[row];
  float x[COLS / 64], px[COLS / 64], dot = 0.f;
#pragma unroll
  for (int k = 0; k < COLS / 64; ++k) {
    const int c = c0 + lane + 64 * k;
    x[k] = c < C ? rz[c] : 0.f;
    px[k] = ce && c < C ? p[c] : 0.f;
  }
  if (ce) {
    float pr[REGS], rr[REGS];
#pragma unroll
    for (int k = 0; k < REGS; ++k) {
      const int c = lane + 64 * k;
      pr[k] = c < C ? p[c] : 0.f; rr[k] = c < C ? rz[c] : 0.f;
    }
    row_columns<REGS>(lane, C, [&](int k, int) { dot += pr[k] * rr[k]; }, [&](int c) { dot += p[c] * rz[c]; });
    dot = wave_sum(dot);
  }
#pragma unroll
  for (int k = 0; k < COLS / 64; ++k) {
    const int c = c0 + lane + 64 * k;
    const T v = from_float<T>(!live || c >= C ? 0.f : ce ? si * (px[k] * x[k] - px[k] * dot) : si * 2.f * x[k]);
    if (live && c < C) D[(long long)row * ldD + c] = v;
    tile[lane + 64 * k][wave] = v;
  }
  store_rows_transposed<ROWS, COLS, T>(tile, Dt, ldDt, i0, c0, C);
}

template <typename T, int REGS>
static void launch_loss_hessian_rows_of(hipStream_t st, int loss, const float* P, const float* Rz, long long ld,
                                        const float* s, int rows, int C, void* D, int ldD, void* Dt, int ldDt) {
  const dim3 grid(lr_up(rows, lr_rows(REGS)), lr_up(C, lr_cols(REGS)));
  loss_hessian_rows_kernel<T, REGS><<<grid, 64 * lr_rows(REGS), 0, st>>>(loss, P, Rz, ld, s, rows, C, (T*)D, ldD, (T*)Dt, ldDt);
}
void launch_loss_hessian_rows(Ctx& ctx, Elem elem, int loss, const float* P, const float* Rz, long long ld,
                              const float* s, int rows, int C, void* D, int ldD, void* Dt, int ldDt) {
  if (rows <= 0) return;
  Launch l(ctx, BETTY_K_LOSS);
  const int regs = lr_regs(C);
  const bool bf = elem == ELEM_BF16;
  auto f = regs == 1 ? (bf ? launch_loss_hessian_rows_of<__bf16, 1> : launch_loss_hessian_rows_of<float, 1>)
         : regs == 4 ? (bf ? launch_loss_hessian_rows_of<__bf16, 4> : launch_loss_hessian_rows_of<float, 4>)
                     : (bf ? launch_loss_hessian_rows_of<__bf16, 16> : launch_loss_hessian_rows_of<float, 16>);
  f(ctx.stream, loss, P, Rz, ld, s, rows, C, D, ldD, Dt, ldDt);
}

__global__ __launch_bounds__(256) void loss_directional_rows_kernel(int loss, const float* P, const float* Z,
                                                                    const Labels* labels, const float* Rz,
                                                                    long long ld, int rows, int C, float* cvec) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float* rz = Rz + (long long)row * ld;
  const Labels lab = *labels;
  float acc = 0.f;
  if (loss == BETTY_LOSS_SOFTMAX_CE) {
    const float* p = P + (long long)row * ld;
    for (int c = lane; c < C; c += 64) acc += p[c] * rz[c];
    acc = wave_sum(acc);
    const int yy = min(max(lab.y[row], 0), C - 1);
    acc -= rz[yy];
  } else {
    const float* z = Z + (long long)row * ld;
    const float* t = lab.target + (long long)row * C;
    for (int c = lane; c < C; c += 64) acc += 2.f * (z[c] - t[c]) * rz[c];
    acc = wave_sum(acc);
  }
  if (lane == 0) cvec[row] = acc;
}

// ------------------------------------------------------------------------------------------
// last layer of the R-op passes for narrow outputs (see LastRopArgs)
// ------------------------------------------------------------------------------------------

// Workgroup = 16 wavefronts, 4 samples.  Both small products run as 16 x 16 MFMA blocks whose rows 4 g + s all hold sample s, so
// that every group of 16 lanes has every sample's results and takes one of them on:
//  phase 1  Rz_L block (4 x C): K = n_in sliced over the wavefronts, partial blocks combined through LDS in wavefront order;
//  phase 2  (one wavefront) loss Hessian per sample with 16-lane butterflies -> R delta_L, kept in
//           LDS in operand type next to delta_L;
//  phase 3  each wavefront takes 16 columns j at a time: R delta_L W^T + delta_L V^T has K = 16 + 16 classes, then the
//           elementwise part, a sample and column a lane, and both output copies.
// SAMPLES: the direction's products come in as AS and DS (a form of its own: fewer registers).
// Deltas and everything beside them are zero beyond the batch and the layers' widths.
// Bound by the one memory round trip and by what the L1 of a compute unit takes in meanwhile.  784-256-10, fp32, batch 128: 4.9 ->
// 2.6 us from first instruction to last (a call of K = 5 119 -> 105 us): 32 x 32 blocks spent 2 us on padding in the matrix cores, and
// loads for rows that hold nothing cost as much as real ones.  3072-1024-1024-1024-10, bf16, batch 256: 5.4 -> 3.6 us.
template <typename T, bool SAMPLES>
__global__ __launch_bounds__(1024) void last_layer_rop_kernel(LastRopArgs a) {
  constexpr int S = 4, CP = LAST_ROP_MAX_C, EPC = 16 / (int)sizeof(T), KS = 4 * EPC, NW = 16, U = 2, NB = 2, HALF = CP / EPC;
  __shared__ float part[NW][S * CP];
  __shared__ __attribute__((aligned(16))) T cat[S][2 * CP];                    // R delta_L, delta_L
  const int t = threadIdx.x, lane = t & 63, ks = __builtin_amdgcn_readfirstlane(t >> 6);
  const int fr = lane & 15, q = lane >> 4;
  // blockIdx.y splits the columns j of phase 3; every split repeats phases 1-2 for its samples
  // (cheap), the first one writes R delta_L
  const int i0 = blockIdx.x * S;
  const int jsplit = ((a.n_in + gridDim.y - 1) / gridDim.y + 15) / 16 * 16;
  const int j_begin = blockIdx.y * jsplit, j_end = a.cvec ? 0 : min(a.n_in, j_begin + jsplit);     // (the directional form has no phase 3)

  // operands of phase 1, the first U steps of this wavefront
  const int steps = (a.n_in + KS - 1) / KS, per = (steps + NW - 1) / NW;
  const int s_begin = min(ks * per, steps), s_end = min(steps, s_begin + per);
  // (Lanes of rows that hold nothing load nothing: what a compute unit's L1 takes in, 16 cycles for 64 lanes' 16 bytes, is
  // what a launch waits for here.)
  const T* const ra = (const T*)a.RA + (long long)(i0 + (fr & 3)) * a.lda + q * EPC;
  const T* const av = (const T*)a.A + (long long)(i0 + (fr & 3)) * a.lda + q * EPC;
  const T* const w = (const T*)a.Wt + (long long)fr * a.ldt + q * EPC;
  const T* const v = (const T*)a.Vt + (long long)fr * a.ldt + q * EPC;
  u32x4 r8[U] = {}, a8[U] = {}, w8[U] = {}, v8[U] = {};
  auto request = [&](int s) {
    if (fr < S) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s_end) {
          r8[u] = *(const u32x4*)(ra + (s + u) * KS);
          if constexpr (!SAMPLES) a8[u] = *(const u32x4*)(av + (s + u) * KS);
        }
    }
    if (fr < a.C) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s_end) {
          w8[u] = *(const u32x4*)(w + (s + u) * KS);
          if constexpr (!SAMPLES) v8[u] = *(const u32x4*)(v + (s + u) * KS);
        }
    }
  };
  request(s_begin);

  // Everything phases 2 and 3 read from memory is independent of phase 1: requested beside its operands and not waited for at its
  // barrier, so the kernel pays one memory round trip (1 to 2 us) instead of three.  (The launcher sizes the column splits so that a wavefront has at most NB blocks of 16 columns.)
  u32x4 w3[NB] = {}, v3[NB] = {};
  float dphi3[NB], e23[NB], rz3[NB], ds3[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int jb = j_begin + (ks + NW * n) * 16;
    dphi3[n] = e23[n] = rz3[n] = ds3[n] = 0.f;
    if (jb >= j_end) break;
    const long long wo = (long long)(jb + fr) * a.ldn;
    if constexpr (sizeof(T) == 2) {
      // one step of 32: chunks 0 and 1 are W with R delta_L, 2 and 3 V with delta_L
      const T* x = (const T*)(!SAMPLES && q >= HALF ? a.Vn : a.Wn) + wo + (q & 1) * EPC;
      w3[n] = *(const u32x4*)x;
    } else {
      w3[n] = *(const u32x4*)((const T*)a.Wn + wo + q * EPC);
      if constexpr (!SAMPLES) v3[n] = *(const u32x4*)((const T*)a.Vn + wo + q * EPC);
    }
    const long long f = (long long)(i0 + q) * a.ldf + jb + fr;
    dphi3[n] = a.dphi[f];
    if (a.e2) { e23[n] = a.e2[f]; rz3[n] = a.Rz[f]; }
    if constexpr (SAMPLES) ds3[n] = a.DS[f];
  }
  float p2 = 0.f, s2 = 0.f, cb2 = 0.f;
  Labels lab{};
  T d2 = from_float<T>(0.f);
  if (ks == 0) {
    const int i = i0 + q;
    if (a.loss == BETTY_LOSS_SOFTMAX_CE) p2 = a.P[(long long)i * a.ldp + fr];
    if constexpr (SAMPLES) cb2 = a.AS[(long long)i * a.ldas + fr];
    else if (a.cbias) cb2 = a.cbias[min(fr, a.C - 1)];
    if (a.cvec) {
      lab = *a.labels;
    } else {
      s2 = a.s[i];
      d2 = ((const T*)a.DL)[(long long)i * a.ldd + fr];
    }
  }

  // ---- phase 1
  MfmaSum16<T> sums;
  for (int s = s_begin; s < s_end; s += U) {
    if (s > s_begin) request(s);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s_end) break;
      sums.step(r8[u], w8[u]);
      if constexpr (!SAMPLES) sums.step(a8[u], v8[u]);
    }
  }
  const f32x4v acc = sums.total();
  if (lane < CP) {
#pragma unroll
    for (int r = 0; r < S; ++r) part[ks][r * CP + lane] = acc[r];
  }
  lds_barrier();

  // ---- phase 2: 16 lanes per sample (lane % 16 = class)
  if (ks == 0) {
    const int i = i0 + q;
    float rz = 0.f;
#pragma unroll
    for (int k = 0; k < NW; ++k) rz += part[k][lane];
    const bool ok = fr < a.C && i < a.B;
    rz = ok ? rz + cb2 : 0.f;
    if (a.cvec) {                                           // directional form: one number per sample
      float term = 0.f;
      if (ok) {
        if (a.loss == BETTY_LOSS_SOFTMAX_CE) {
          const int yy = min(max(lab.y[i], 0), a.C - 1);
          term = p2 * rz - (fr == yy ? rz : 0.f);
        } else {
          term = 2.f * (a.Z[(long long)i * a.ldp + fr] - lab.target[(long long)i * a.C + fr]) * rz;
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) term += __shfl_xor(term, o, 64);
      if (fr == 0 && i < a.B) a.cvec[i] = term;
    } else {
      float val;
      if (a.loss == BETTY_LOSS_SOFTMAX_CE) {
        float dot = p2 * rz;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) dot += __shfl_xor(dot, o, 64);
        val = s2 * (p2 * rz - p2 * dot);
      } else {
        val = s2 * 2.f * rz;
      }
      const T vt = from_float<T>(ok ? val : 0.f);
      cat[q][fr] = vt;
      cat[q][CP + fr] = SAMPLES ? from_float<T>(0.f) : d2;
      if (ok && blockIdx.y == 0) {
        ((T*)a.RDL)[(long long)i * a.ldd + fr] = vt;
        ((T*)a.RDLt)[(long long)fr * a.ldRDLt + i] = vt;
      }
    }
  }
  lds_barrier();                                            // (every wavefront reaches this, in both forms)

  // ---- phase 3
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int jb = j_begin + (ks + NW * n) * 16, j = jb + fr, i = i0 + q;
    if (jb >= j_end) continue;
    f32x4v o4 = {0.f, 0.f, 0.f, 0.f};
    const T* c = &cat[fr & 3][q * EPC];
    MfmaStep16<T>::run(*(const u32x4*)c, w3[n], o4);
    if constexpr (sizeof(T) == 4 && !SAMPLES) MfmaStep16<T>::run(*(const u32x4*)(c + CP), v3[n], o4);
    // register s of every lane: sample s of column j; this lane takes sample q
    float o = q == 0 ? o4[0] : q == 1 ? o4[1] : q == 2 ? o4[2] : o4[3];
    o = i < a.B ? (SAMPLES ? o + ds3[n] : o) * dphi3[n] + e23[n] * rz3[n] : 0.f;     // rows beyond the batch: zero padding
    if (j >= j_end) continue;
    if (a.RD && i < a.B) ((T*)a.RD)[(long long)i * a.ldRD + j] = from_float<T>(o);
    ((T*)a.RDt)[(long long)j * a.ldRDt + i] = from_float<T>(o);
  }
}

void launch_last_layer_rop(Ctx& ctx, Elem elem, const LastRopArgs& a) {
  if (a.B <= 0) return;
  Launch l(ctx, BETTY_K_LAST_LAYER, 8.0 * a.B * a.n_in * a.C, 0);      // two pairs in each of two products
  const int blocks = (a.B + 3) / 4;
  // column splits: at most two blocks of 16 columns per wavefront (512 columns per workgroup), and
  // enough workgroups to occupy the chip
  const int splits = a.cvec ? 1 : std::max((a.n_in + 511) / 512, std::max(1, std::min(256 / blocks, (a.n_in + 31) / 32)));
  const dim3 grid(blocks, splits);
  if (elem == ELEM_BF16) {
    if (a.AS) last_layer_rop_kernel<__bf16, true><<<grid, 1024, 0, ctx.stream>>>(a);
    else last_layer_rop_kernel<__bf16, false><<<grid, 1024, 0, ctx.stream>>>(a);
  } else {
    if (a.AS) last_layer_rop_kernel<float, true><<<grid, 1024, 0, ctx.stream>>>(a);
    else last_layer_rop_kernel<float, false><<<grid, 1024, 0, ctx.stream>>>(a);
  }
}

// Same layout as last_layer_rop_kernel (16 wavefronts, 4 samples, 16 x 16 MFMA blocks);
// blockIdx.z selects the batch.
template <typename T>
__global__ __launch_bounds__(1024) void last_layer_grad_kernel(LastGradArgs a) {
  constexpr int S = 4, CP = LAST_ROP_MAX_C, EPC = 16 / (int)sizeof(T), KS = 4 * EPC, NW = 16, U = 2, NB = 2, HALF = CP / EPC;
  __shared__ float part[NW][S * CP];
  __shared__ __attribute__((aligned(16))) T dlT[S][2 * CP];                    // (bf16: a step of 32, whose second half is zero)
  const LastGradSide& sd = a.side[blockIdx.z];
  const int t = threadIdx.x, lane = t & 63, ks = __builtin_amdgcn_readfirstlane(t >> 6);
  const int fr = lane & 15, g = lane >> 4;
  const int i0 = blockIdx.x * S;
  if (i0 >= sd.B) return;                                   // the two batches may differ in size
  const int jsplit = ((a.n_in + gridDim.y - 1) / gridDim.y + 15) / 16 * 16;
  const int j_begin = blockIdx.y * jsplit, j_end = min(a.n_in, j_begin + jsplit);

  // operands of phase 1, the first U steps of this wavefront
  const int steps = (a.n_in + KS - 1) / KS, per = (steps + NW - 1) / NW;
  const int s_begin = min(ks * per, steps), s_end = min(steps, s_begin + per);
  const T* const av = (const T*)sd.A + (long long)(i0 + (fr & 3)) * sd.lda + g * EPC;
  const T* const w = (const T*)sd.Wt + (long long)fr * a.ldt + g * EPC;
  u32x4 a8[U] = {}, w8[U] = {};
  auto request = [&](int s) {
    if (fr < S) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s_end) a8[u] = *(const u32x4*)(av + (s + u) * KS);
    }
    if (fr < a.C) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < s_end) w8[u] = *(const u32x4*)(w + (s + u) * KS);
    }
  };
  request(s_begin);

  // inputs of phase 3 that do not depend on the earlier phases
  u32x4 w3[NB] = {};
  float dphi3[NB], e23[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int jb = j_begin + (ks + NW * n) * 16;
    dphi3[n] = e23[n] = 0.f;
    if (jb >= j_end) break;
    if (g < HALF) w3[n] = *(const u32x4*)((const T*)sd.Wn + (long long)(jb + fr) * a.ldn + g * EPC);
    const long long f = (long long)(i0 + g) * sd.ldf + jb + fr;
    dphi3[n] = sd.dphi[f];
    if (sd.e2) e23[n] = sd.e2[f];
  }

  // ... and the label (or target) and bias of phase 2
  float t2 = 0.f, bias2 = 0.f;
  int y2 = 0;
  if (ks == 0) {
    const int i = i0 + g;
    const Labels lab = *sd.labels;
    if (i < sd.B) {
      if (a.loss == BETTY_LOSS_SOFTMAX_CE) y2 = lab.y[i];
      else if (fr < a.C) t2 = lab.target[(long long)i * a.C + fr];
      if (fr < a.C && sd.bias) bias2 = sd.bias[fr];
    }
  }

  // ---- phase 1: logits block (4 x C), K = n_in sliced over the wavefronts
  MfmaSum16<T> sums;
  for (int s = s_begin; s < s_end; s += U) {
    if (s > s_begin) request(s);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s_end) break;
      sums.step(a8[u], w8[u]);
    }
  }
  const f32x4v acc = sums.total();
  if (lane < CP) {
#pragma unroll
    for (int r = 0; r < S; ++r) part[ks][r * CP + lane] = acc[r];
  }
  lds_barrier();

  // ---- phase 2: 16 lanes per sample (lane % 16 = class)
  if (ks == 0) {
    const int s = lane >> 4, c = lane & 15, i = i0 + s;
    const bool iok = i < sd.B, ok = iok && c < a.C;
    float z = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) z += part[q][lane];
    z += bias2;
    float ell, p = 0.f, dz;
    int y = 0;
    if (a.loss == BETTY_LOSS_SOFTMAX_CE) {
      float m = ok ? z : -INFINITY;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      const float ex = ok ? expf(z - m) : 0.f;
      float sum = ex;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
      y = min(max(y2, 0), a.C - 1);      // clamped into [0, C), for the gather and the one-hot alike
      const float zy = __shfl(z, (lane & ~15) + y, 64);
      ell = logf(sum) + m - zy;
      p = ex / sum;
      dz = p - (c == y ? 1.f : 0.f);
    } else {
      const float r = ok ? z - t2 : 0.f;
      float acc2 = r * r;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) acc2 += __shfl_xor(acc2, o, 64);
      ell = acc2;
      dz = 2.f * r;
    }
    float omega = 1.f;
    if (sd.reweight && sd.omega_fixed) {
      omega = iok ? sd.omega_fixed[i] : 1.f;
    } else if (sd.reweight) {
      const int H = a.hidden;
      float pw = 0.f;
      for (int hj = c; hj < H; hj += 16) pw += a.theta[2 * H + hj] * fmaxf(a.theta[hj] * ell + a.theta[H + hj], 0.f);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) pw += __shfl_xor(pw, o, 64);
      const float logit = pw + a.theta[3 * H];
      omega = 1.f / (1.f + expf(-logit));
      if (blockIdx.y == 0 && iok && c == 0 && sd.dsig) sd.dsig[i] = omega / (1.f + expf(logit));
    }
    const float sc = omega * sd.inv_batch;
    const T dv = from_float<T>(sc * dz);
    dlT[s][c] = ok ? dv : from_float<T>(0.f);
    dlT[s][CP + c] = from_float<T>(0.f);
    if (blockIdx.y == 0) {
      if (iok && c == 0) { sd.ell[i] = ell; sd.s[i] = sc; sd.omega[i] = omega; }
      if (ok) {
        sd.ZL[(long long)i * sd.ldz + c] = z;
        if (a.loss == BETTY_LOSS_SOFTMAX_CE) sd.P[(long long)i * sd.ldz + c] = p;
        ((T*)sd.DL)[(long long)i * sd.ldd + c] = dv;
        ((T*)sd.DLt)[(long long)c * sd.ldDLt + i] = dv;
      }
    }
  }
  lds_barrier();

  // ---- phase 3: delta_{L-1}, 16 columns a block; rows 4 g + s of a block all hold sample s, and a lane takes sample g on
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int jb = j_begin + (ks + NW * n) * 16, j = jb + fr, i = i0 + g;
    if (jb >= j_end) break;
    f32x4v o4 = {0.f, 0.f, 0.f, 0.f};
    MfmaStep16<T>::run(*(const u32x4*)&dlT[fr & 3][g * EPC], w3[n], o4);
    const float o = g == 0 ? o4[0] : g == 1 ? o4[1] : g == 2 ? o4[2] : o4[3];
    if (j >= j_end) continue;
    const bool iok = i < sd.B;
    const float dl = iok ? o * dphi3[n] : 0.f;              // rows beyond the batch: zero padding
    if (iok && sd.D) ((T*)sd.D)[(long long)i * sd.ldD + j] = from_float<T>(dl);
    if (iok && sd.e2) sd.e2[(long long)i * sd.ldf + j] = o * e23[n];
    ((T*)sd.Dt)[(long long)j * sd.ldDt + i] = from_float<T>(dl);
  }
}

void launch_last_layer_grad(Ctx& ctx, Elem elem, const LastGradArgs& a) {
  int blocks = 0;
  for (int i = 0; i < a.n_sides; ++i) blocks = std::max(blocks, (a.side[i].B + 3) / 4);
  if (blocks <= 0) return;
  double flops = 0;
  for (int i = 0; i < a.n_sides; ++i) flops += 4.0 * a.side[i].B * a.n_in * a.C;
  Launch l(ctx, BETTY_K_LAST_LAYER, flops, 0);
  const int splits = std::max((a.n_in + 511) / 512, std::max(1, std::min(256 / (blocks * a.n_sides), (a.n_in + 31) / 32)));
  const dim3 grid(blocks, splits, a.n_sides);
  if (elem == ELEM_BF16) last_layer_grad_kernel<__bf16><<<grid, 1024, 0, ctx.stream>>>(a);
  else last_layer_grad_kernel<float><<<grid, 1024, 0, ctx.stream>>>(a);
}

void launch_loss_directional_rows(Ctx& ctx, int loss, const float* P, const float* Z, const Labels* labels,
                                  const float* Rz, long long ld, int rows, int C, float* c) {
  if (rows <= 0) return;
  Launch l(ctx, BETTY_K_LOSS);
  loss_directional_rows_kernel<<<(rows + 3) / 4, 256, 0, ctx.stream>>>(loss, P, Z, labels, Rz, ld, rows, C, c);
}

// one block per hidden unit (and one for the output bias): fixed-order sums over the samples
__global__ __launch_bounds__(256) void wnet_theta_vjp_kernel(const float* ell, const float* dsig,
                                                             const float* cvec, const float* cminus, const float* eps,
                                                             const float* theta, int H, int rows, float inv_batch,
                                                             float* out) {
  __shared__ float red[4];
  const int j = blockIdx.x;
  const float e = cminus ? eps[0] : 0.f;
  auto ci = [&](int i) { return !cminus ? cvec[i] : e > 0.f ? (cvec[i] - cminus[i]) / (2.f * e) : 0.f; };
  float a1 = 0.f, a2 = 0.f, a3 = 0.f;
  if (j < H) {
    const float u1 = theta[j], b1 = theta[H + j], u2 = theta[2 * H + j];
    for (int i = threadIdx.x; i < rows; i += 256) {
      const float ds = ci(i) * dsig[i];
      const float pre = u1 * ell[i] + b1;
      const float on = pre > 0.f ? 1.f : 0.f;
      a1 += ds * u2 * on * ell[i];
      a2 += ds * u2 * on;
      a3 += ds * fmaxf(pre, 0.f);
    }
    a1 = block_sum(a1, red); a2 = block_sum(a2, red); a3 = block_sum(a3, red);
    if (threadIdx.x == 0) {
      out[j] = -inv_batch * a1; out[H + j] = -inv_batch * a2; out[2 * H + j] = -inv_batch * a3;
    }
  } else {
    for (int i = threadIdx.x; i < rows; i += 256) a1 += ci(i) * dsig[i];
    a1 = block_sum(a1, red);
    if (threadIdx.x == 0) out[3 * H] = -inv_batch * a1;
  }
}

void launch_wnet_theta_vjp(Ctx& ctx, const float* ell, const float* dsig, const float* c, const float* c_minus, const float* eps,
                           const float* theta, int hidden, int rows, float inv_batch, float* out) {
  Launch l(ctx, BETTY_K_WNET);
  wnet_theta_vjp_kernel<<<hidden + 1, 256, 0, ctx.stream>>>(ell, dsig, c, c_minus, eps, theta, hidden, rows, inv_batch, out);
}

// ------------------------------------------------------------------------------------------
// streaming kernels over flat vectors
// ------------------------------------------------------------------------------------------

static inline unsigned flat_grid(size_t n) {
  size_t b = (n + 255) / 256;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (unsigned)b;
}

#define FLAT_LOOP(i, n) \
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < (n); i += (size_t)gridDim.x * 256)

__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* p, size_t n16) {
  FLAT_LOOP(i, n16) p[i] = make_uint4(0, 0, 0, 0);
}
void launch_fill_zero(Ctx& ctx, void* p, size_t bytes) {
  if (!bytes) return;
  Launch l(ctx, BETTY_K_OTHER, 0, (double)bytes);
  fill_zero_kernel<<<flat_grid(bytes / 16), 256, 0, ctx.stream>>>((uint4*)p, bytes / 16);
}

template <bool FD>
__global__ __launch_bounds__(256) void mixed_l2_kernel(const float* lam, const float* w, const float* p, float alpha, float* out, size_t n) {
  FLAT_LOOP(i, n) out[i] = FD ? fd_mixed_l2(lam[i], w[i], alpha, p[i]) : -2.f * expf(lam[i]) * w[i] * (alpha * p[i]);
}
void launch_mixed_l2(Ctx& ctx, const float* lam, const float* w, const float* p, float alpha, float* out, size_t n, bool fd) {
  Launch l(ctx, BETTY_K_VECTOR, 0, 16.0 * n);
  if (fd) mixed_l2_kernel<true><<<flat_grid(n), 256, 0, ctx.stream>>>(lam, w, p, alpha, out, n);
  else mixed_l2_kernel<false><<<flat_grid(n), 256, 0, ctx.stream>>>(lam, w, p, alpha, out, n);
}

__global__ __launch_bounds__(256) void mixed_prox_kernel(const float* logrho, const float* p, float alpha, float* out, size_t n) {
  FLAT_LOOP(i, n) out[i] = 2.f * expf(logrho[i]) * (alpha * p[i]);
}
void launch_mixed_prox(Ctx& ctx, const float* logrho, const float* p, float alpha, float* out, size_t n) {
  Launch l(ctx, BETTY_K_VECTOR, 0, 12.0 * n);
  mixed_prox_kernel<<<flat_grid(n), 256, 0, ctx.stream>>>(logrho, p, alpha, out, n);
}

__global__ __launch_bounds__(256) void fill_value_kernel(float* p, float value, size_t n) {
  FLAT_LOOP(i, n) p[i] = value;
}
void launch_fill_value(Ctx& ctx, float* p, float value, size_t n) {
  if (n == 0) return;
  Launch l(ctx, BETTY_K_VECTOR, 0, 4.0 * n);
  fill_value_kernel<<<flat_grid(n), 256, 0, ctx.stream>>>(p, value, n);
}

// Adam on the upper parameters: bias1 = 1 - beta1^t, bias2 = 1 - beta2^t are formed on the host
__global__ __launch_bounds__(256) void adam_kernel(float* x, const float* g, float* m, float* v, float lr, float beta1,
                                                   float beta2, float eps, float bias1, float bias2, size_t n) {
  FLAT_LOOP(i, n) {
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    x[i] -= lr * (mi / bias1) / (sqrtf(vi / bias2) + eps);
  }
}
void launch_adam(Ctx& ctx, float* x, const float* g, float* m, float* v, float lr, float beta1, float beta2, float eps,
                 float bias1, float bias2, size_t n) {
  Launch l(ctx, BETTY_K_VECTOR, 0, 28.0 * n);
  adam_kernel<<<flat_grid(n), 256, 0, ctx.stream>>>(x, g, m, v, lr, beta1, beta2, eps, bias1, bias2, n);
}

// the sums that weight-gradient launches leave behind (16-byte aligned): one block, fixed order
template <int NT>
__device__ __forceinline__ double sum_partials(const double* p, int n, double* red) {
  double acc = 0.0;
  const int n2 = n / 2;
  for (int i = threadIdx.x; i < n2; i += NT) {
    const double2 x = ((const double2*)p)[i];
    acc += x.x + x.y;
  }
  if (threadIdx.x == 0 && n > 2 * n2) acc += p[n - 1];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) t += red[k];
  return t;
}

__global__ __launch_bounds__(1024) void weighted_loss_sum_kernel(const float* s, const float* ell, int rows, const double* partial, int n, float* out) {
  __shared__ double red[16], red2[16];
  const double cost = sum_partials<1024>(partial, n, red2);
  double acc = 0.0;
  for (int i = threadIdx.x; i < rows; i += 1024) acc += (double)s[i] * (double)ell[i];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t = 0.0;
  for (int k = 0; k < 16; ++k) t += red[k];
  out[0] = (float)(t + cost);
}
void launch_weighted_loss_sum(Ctx& ctx, const float* s, const float* ell, int rows, const double* partial, int n, float* out) {
  Launch l(ctx, BETTY_K_REDUCE);
  weighted_loss_sum_kernel<<<1, 1024, 0, ctx.stream>>>(s, ell, rows, partial, n, out);
}

__device__ __forceinline__ float fd_step(double sumsq, float eps_scale, float scale) {
  const float nrm = sqrtf((float)sumsq) * fabsf(scale);
  return nrm > 0.f ? eps_scale / nrm : 0.f;
}
__global__ __launch_bounds__(1024) void fd_eps_kernel(const double* partial, int n, float eps_scale, float scale, float* eps) {
  __shared__ double red[16];
  const double s = sum_partials<1024>(partial, n, red);
  if (threadIdx.x == 0) eps[0] = fd_step(s, eps_scale, scale);
}
void launch_fd_eps(Ctx& ctx, const double* partial, int n, float eps_scale, float scale, float* eps) {
  Launch l(ctx, BETTY_K_OTHER, 0, 8.0 * n);
  fd_eps_kernel<<<1, 1024, 0, ctx.stream>>>(partial, n, eps_scale, scale, eps);
}

// ---- conjugate gradient (scalars stay on the device; nothing here reads them on the host)
//
// Bound by the launches for small problems: every block adds up the partial sums of the launch before
// it again, in the same order (a few KB out of L2), instead of a launch between that leaves one number, and the
// new direction leaves as GEMM operands.  Two launches a step where there were six (784 x 10 parameters: 28 -> 19
// us a step with the Hessian product).
constexpr int CG_BLOCKS = 1024;

__global__ __launch_bounds__(256) void cg_step_kernel(CgStep c) {
  __shared__ double red[4], red2[4];
  const float den = (float)sum_partials<256>(c.dHd, c.n_dHd, red);
  float num;
  if (c.rs_partial) {
    num = (float)sum_partials<256>(c.rs_partial, c.n_rs, red2);
    if (blockIdx.x == 0 && threadIdx.x == 0) *c.rs = num;
  } else {
    num = *c.rs;
  }
  const float a = (num != 0.f && den != 0.f) ? num / den : 0.f;
  if (c.out) {
    FLAT_LOOP(i, c.n) {
      const float qi = (c.rs_partial ? 0.f : c.q[i]) + a * c.d[i], el = 2.f * expf(c.lam[i]);
      c.out[i] = c.w ? -el * c.w[i] * qi : el * qi;
    }
    return;
  }
  float acc = 0.f;
  double dacc = 0.0;
  int cnt = 0;
  FLAT_LOOP(i, c.n) {
    c.q[i] = (c.rs_partial ? 0.f : c.q[i]) + a * c.d[i];
    const float ri = c.r[i] - a * c.Hd[i];
    c.r[i] = ri;
    acc += ri * ri;
    if (++cnt == 64) { dacc += acc; acc = 0.f; cnt = 0; }
  }
  dacc += acc;
  dacc = block_sum(dacc, red);
  if (threadIdx.x == 0) c.partials[blockIdx.x] = dacc;
}
int launch_cg_step(Ctx& ctx, const CgStep& c) {
  const unsigned nb = std::min<unsigned>(flat_grid(c.n), CG_BLOCKS);
  Launch l(ctx, BETTY_K_VECTOR, 0, 24.0 * c.n);
  cg_step_kernel<<<nb, 256, 0, ctx.stream>>>(c);
  return (int)nb;
}

template <typename T>
__global__ __launch_bounds__(256) void cg_dir_kernel(CgDirBatch b) {
  __shared__ float tile[64][65];
  __shared__ double red[4];
  int bid = blockIdx.x, ji = 0;
  while (ji + 1 < b.n && bid >= b.block_begin[ji + 1]) ++ji;
  const CgDirJob& j = b.j[ji];
  bid -= b.block_begin[ji];
  const int tiles_x = (j.cols + 63) / 64;
  const int c0 = (bid % tiles_x) * 64, r0 = (bid / tiles_x) * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, c = c0 + 4 * tx;
  const bool quads = j.cols % 4 == 0 && ((uintptr_t)j.r & 15) == 0 && ((uintptr_t)j.d & 15) == 0;
  float r[4][4], d[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const long long row = (long long)min(r0 + ty + 16 * i, j.rows - 1) * j.cols;
    if (quads) {
      const long long at = row + min(c, j.cols - 4);
      const float4 x = *(const float4*)(j.r + at), y = *(const float4*)(j.d + at);
      r[i][0] = x.x; r[i][1] = x.y; r[i][2] = x.z; r[i][3] = x.w;
      d[i][0] = y.x; d[i][1] = y.y; d[i][2] = y.z; d[i][3] = y.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const long long at = row + min(c + k, j.cols - 1);
        r[i][k] = j.r[at]; d[i][k] = j.d[at];
      }
    }
  }
  const float rs = *b.rs;
  double acc = 0.0;
  for (int i = threadIdx.x; i < b.n_partial; i += 256) acc += b.partials[i];
  const float rs_new = (float)block_sum(acc, red), beta = rs != 0.f ? rs_new / rs : 0.f;
  if (blockIdx.x == 0 && ji == 0 && threadIdx.x == 0 && b.rs_new) *b.rs_new = rs_new;
  if (j.bd && r0 == 0 && threadIdx.x < 64 && c0 + (int)threadIdx.x < j.cols) {     // biases: with the first row of tiles
    const int cb = c0 + threadIdx.x;
    j.bd[cb] = j.br[cb] + beta * j.bd[cb];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = ty + 16 * i, row = r0 + rl;
    float x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { x[k] = r[i][k] + beta * d[i][k]; tile[rl][4 * tx + k] = x[k]; }
    if (row >= j.rows) continue;
    float* o = j.d + (long long)row * j.cols + c;
    T* p = (T*)j.out + (long long)row * j.ld + c;              // (operands: pitch a multiple of 128, 256-byte aligned)
    if (c + 3 < j.cols) {
      if (quads) *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
      else
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = x[k];
      if (j.out) store_quad<T>(p, x[0], x[1], x[2], x[3]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) if (c + k < j.cols) { o[k] = x[k]; if (j.out) p[k] = from_float<T>(x[k]); }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int cl = ty + 16 * i, cc = c0 + cl, row = r0 + 4 * tx;
    if (cc >= j.cols || row >= j.rows) continue;
    T* o = (T*)j.outT + (long long)cc * j.ldT + row;
    const float x[4] = {tile[4 * tx][cl], tile[4 * tx + 1][cl], tile[4 * tx + 2][cl], tile[4 * tx + 3][cl]};
    if (row + 3 < j.rows) store_quad<T>(o, x[0], x[1], x[2], x[3]);
    else
#pragma unroll
      for (int k = 0; k < 4; ++k) if (row + k < j.rows) o[k] = from_float<T>(x[k]);
  }
}
void launch_cg_dir(Ctx& ctx, Elem elem, CgDirBatch& b) {
  int blocks = 0;
  double params = 0;
  for (int i = 0; i < b.n; ++i) {
    b.block_begin[i] = blocks;
    blocks += ((b.j[i].cols + 63) / 64) * ((b.j[i].rows + 63) / 64);
    params += (double)b.j[i].rows * b.j[i].cols;
  }
  b.block_begin[b.n] = blocks;
  if (blocks <= 0) return;
  Launch l(ctx, BETTY_K_VECTOR, 0, (12.0 + 2.0 * elem_size(elem)) * params);
  if (elem == ELEM_BF16) cg_dir_kernel<__bf16><<<blocks, 256, 0, ctx.stream>>>(b);
  else cg_dir_kernel<float><<<blocks, 256, 0, ctx.stream>>>(b);
}

// cg_step and cg_dir in one launch.  Few parameters: a workgroup reads both vectors for the sum, 64 KB of 8 000 parameters,
// sooner than another launch would start (784 x 10, batch 512, K = 8: 152 -> 132 us a call).
template <typename T>
__global__ __launch_bounds__(1024) void cg_update_kernel(CgUpdate b) {
  __shared__ float tile[64][65];
  __shared__ double red[16], red2[16], red3[16];
  const int t = threadIdx.x;
  int bid = blockIdx.x, ji = 0;
  while (ji + 1 < b.n && bid >= b.block_begin[ji + 1]) ++ji;
  const CgUpdateJob& j = b.j[ji];
  bid -= b.block_begin[ji];
  const int tiles_x = (j.cols + 63) / 64, c0 = (bid % tiles_x) * 64, r0 = (bid / tiles_x) * 64;
  // the tile's own elements: four rows 16 apart of one column
  const int tx = t & 63, ty = t >> 6, c = min(c0 + tx, j.cols - 1);
  float r[4], h[4], d[4], q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const long long at = j.at + (long long)min(r0 + ty + 16 * i, j.rows - 1) * j.cols + c;
    r[i] = b.r[at]; h[i] = b.Hd[at]; d[i] = b.d[at]; q[i] = b.rs_partial ? 0.f : b.q[at];
  }
  // all of the residual (the vectors stand at multiples of 256 bytes); at most CG_ONE / 4096 quads a thread
  constexpr int QUADS = CG_ONE / 4096;
  const int quads = b.params >> 2;
  float4 fr[QUADS], fh[QUADS];
#pragma unroll
  for (int i = 0; i < QUADS; ++i) {
    if (i * 1024 >= quads) break;
    const int x = min(t + 1024 * i, quads - 1);
    fr[i] = ((const float4*)b.r)[x]; fh[i] = ((const float4*)b.Hd)[x];
  }
  const int rest = 4 * quads + t;
  const bool has_rest = rest < b.params;
  const float rr = has_rest ? b.r[rest] : 0.f, rh = has_rest ? b.Hd[rest] : 0.f;
  const float den = (float)sum_partials<1024>(b.dHd, b.n_dHd, red);
  const float num = b.rs_partial ? (float)sum_partials<1024>(b.rs_partial, b.n_rs, red2) : *b.rs;
  const float a = (num != 0.f && den != 0.f) ? num / den : 0.f;
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < QUADS; ++i) {
    if (i * 1024 >= quads) break;
    const float x0 = fr[i].x - a * fh[i].x, x1 = fr[i].y - a * fh[i].y, x2 = fr[i].z - a * fh[i].z, x3 = fr[i].w - a * fh[i].w;
    if (t + 1024 * i < quads) acc += (double)(x0 * x0 + x1 * x1 + x2 * x2 + x3 * x3);
  }
  const float xr = rr - a * rh;
  if (has_rest) acc += (double)(xr * xr);
  acc = wave_sum(acc);
  if ((t & 63) == 0) red3[t >> 6] = acc;
  __syncthreads();
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) sum += red3[k];
  const float rs_new = (float)sum, beta = num != 0.f ? rs_new / num : 0.f;
  if (blockIdx.x == 0 && t == 0) *b.rs_new = rs_new;
  if (j.bias >= 0 && r0 == 0 && t < 64 && c0 + t < j.cols) {          // biases: with the first row of tiles
    const long long at = j.bias + c0 + t;
    const float db = b.d[at], rb = b.r[at] - a * b.Hd[at];
    b.q[at] = (b.rs_partial ? 0.f : b.q[at]) + a * db;
    b.r_out[at] = rb;
    b.d[at] = rb + beta * db;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rl = ty + 16 * i, row = r0 + rl;
    const float rn = r[i] - a * h[i], x = rn + beta * d[i];
    tile[rl][tx] = x;
    if (row >= j.rows || c0 + tx >= j.cols) continue;
    const long long at = j.at + (long long)row * j.cols + c;
    b.q[at] = q[i] + a * d[i];
    b.r_out[at] = rn;
    b.d[at] = x;
    if (j.out) ((T*)j.out)[(long long)row * j.ld + c] = from_float<T>(x);
  }
  __syncthreads();
  const int cl = t >> 4, r4 = 4 * (t & 15), cc = c0 + cl, row = r0 + r4;
  if (cc >= j.cols || row >= j.rows) return;
  T* const o = (T*)j.outT + (long long)cc * j.ldT + row;
  const float x[4] = {tile[r4][cl], tile[r4 + 1][cl], tile[r4 + 2][cl], tile[r4 + 3][cl]};
  if (row + 3 < j.rows) store_quad<T>(o, x[0], x[1], x[2], x[3]);
  else
#pragma unroll
    for (int k = 0; k < 4; ++k) if (row + k < j.rows) o[k] = from_float<T>(x[k]);
}
void launch_cg_update(Ctx& ctx, Elem elem, CgUpdate& b) {
  int blocks = 0;
  for (int i = 0; i < b.n; ++i) {
    b.block_begin[i] = blocks;
    blocks += ((b.j[i].cols + 63) / 64) * ((b.j[i].rows + 63) / 64);
  }
  b.block_begin[b.n] = blocks;
  if (blocks <= 0) return;
  Launch l(ctx, BETTY_K_VECTOR, 0, (24.0 + 2.0 * elem_size(elem)) * b.params);
  if (elem == ELEM_BF16) cg_update_kernel<__bf16><<<blocks, 1024, 0, ctx.stream>>>(b);
  else cg_update_kernel<float><<<blocks, 1024, 0, ctx.stream>>>(b);
}

// The two perturbed points of a central difference, straight into GEMM operands: w and v are read once,
// 24 bytes a parameter against 48 for two passes of perturbation and conversion each.  64 x 64 tiles as in
// convert_batch_kernel, all loads of a tile in flight together.  EPS: the step comes out of the partial sums
// of |v|^2 in every block, in the same order, beside the loads of the tile, instead of a launch between
// (see fd_seq).
template <bool EPS, int NT>
__global__ __launch_bounds__(NT) void perturb_kernel(PerturbBatch b) {
  constexpr int Q = 1024 / NT, QS = NT / 16;       // quads a thread, their distance in rows
  __shared__ float tile[64][65];
  __shared__ double red[NT / 64];
  int bid = blockIdx.x, ji = 0;
  while (ji + 1 < b.n && bid >= b.block_begin[ji + 1]) ++ji;
  const PerturbJob& j = b.j[ji];
  bid -= b.block_begin[ji];
  const int tiles_x = (j.cols + 63) / 64;
  const int c0 = (bid % tiles_x) * 64, r0 = (bid / tiles_x) * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const bool quads = j.cols % 4 == 0 && ((uintptr_t)j.w & 15) == 0 && ((uintptr_t)j.v & 15) == 0;
  float w[Q][4], v[Q][4];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const long long row = (long long)min(r0 + ty + QS * i, j.rows - 1) * j.cols;
    if (quads) {
      const long long at = row + min(c0 + 4 * tx, j.cols - 4);
      const float4 a = *(const float4*)((j.w ? j.w : j.v) + at), d = *(const float4*)(j.v + at);
      w[i][0] = a.x; w[i][1] = a.y; w[i][2] = a.z; w[i][3] = a.w;
      v[i][0] = d.x; v[i][1] = d.y; v[i][2] = d.z; v[i][3] = d.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const long long at = row + min(c0 + 4 * tx + k, j.cols - 1);
        w[i][k] = (j.w ? j.w : j.v)[at]; v[i][k] = j.v[at];
      }
    }
  }
  float eps;
  if constexpr (EPS) {
    eps = fd_step(sum_partials<NT>(b.partial, b.n_partial, red), b.eps_scale, b.scale);
    if (blockIdx.x == 0 && threadIdx.x == 0) b.eps_out[0] = eps;
  } else {
    eps = b.eps[0];
  }
  if (!j.w) {                                      // the direction itself, transposed
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) tile[ty + QS * i][4 * tx + k] = v[i][k];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int cl = ty + QS * i, c = c0 + cl, r = r0 + 4 * tx;
      if (c >= j.cols) continue;
      float* o = j.outT[0] + (long long)c * j.ldT + r;
      const float x[4] = {tile[4 * tx][cl], tile[4 * tx + 1][cl], tile[4 * tx + 2][cl], tile[4 * tx + 3][cl]};
      if (r + 3 < j.rows) *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
      else
#pragma unroll
        for (int k = 0; k < 4; ++k) if (r + k < j.rows) o[k] = x[k];
    }
    return;
  }
  // biases ride along with the first row of tiles
  if (j.b && r0 == 0 && threadIdx.x < 64 && c0 + (int)threadIdx.x < j.cols) {
    const int c = c0 + threadIdx.x;
    const float bw = j.b[c], bd = b.scale * j.bv[c];
    if (b.signs & 1) j.bout[0][c] = bw + eps * bd;
    if (b.signs & 2) j.bout[1][c] = bw - eps * bd;
  }
#pragma unroll
  for (int sg = 0; sg < 2; ++sg) {
    if (!(b.signs >> sg & 1)) continue;
    const float e = sg ? -eps : eps;
    if (sg && (b.signs & 1)) __syncthreads();       // the tile of the other sign is read out
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int rl = ty + QS * i, r = r0 + rl, c = c0 + 4 * tx;
      float x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { x[k] = w[i][k] + e * (b.scale * v[i][k]); tile[rl][4 * tx + k] = x[k]; }
      if (r < j.rows && j.out[sg]) {
        float* o = j.out[sg] + (long long)r * j.ld + c;      // (ld is a multiple of 128, out 256-byte aligned)
        if (c + 3 < j.cols) *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
        else
#pragma unroll
          for (int k = 0; k < 4; ++k) if (c + k < j.cols) o[k] = x[k];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int cl = ty + QS * i, c = c0 + cl, r = r0 + 4 * tx;
      if (c >= j.cols) continue;
      float* o = j.outT[sg] + (long long)c * j.ldT + r;
      const float x[4] = {tile[4 * tx][cl], tile[4 * tx + 1][cl], tile[4 * tx + 2][cl], tile[4 * tx + 3][cl]};
      if (r + 3 < j.rows) *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
      else
#pragma unroll
        for (int k = 0; k < 4; ++k) if (r + k < j.rows) o[k] = x[k];
    }
  }
}
void launch_perturb(Ctx& ctx, PerturbBatch& b) {
  int blocks = 0;
  double params = 0;
  for (int i = 0; i < b.n; ++i) {
    b.block_begin[i] = blocks;
    blocks += ((b.j[i].cols + 63) / 64) * ((b.j[i].rows + 63) / 64);
    params += (double)b.j[i].rows * b.j[i].cols * (b.j[i].w ? 8.0 + 8.0 * ((b.signs & 1) + (b.signs >> 1)) : 8.0);
  }
  b.block_begin[b.n] = blocks;
  if (blocks <= 0) return;
  Launch l(ctx, BETTY_K_SHADOW, 0, params);
  const bool wide = blocks <= CONVERT_WIDE;
  if (b.eps) {
    if (wide) perturb_kernel<false, 1024><<<blocks, 1024, 0, ctx.stream>>>(b);
    else perturb_kernel<false, 256><<<blocks, 256, 0, ctx.stream>>>(b);
  } else {
    if (wide) perturb_kernel<true, 1024><<<blocks, 1024, 0, ctx.stream>>>(b);
    else perturb_kernel<true, 256><<<blocks, 256, 0, ctx.stream>>>(b);
  }
}

__global__ __launch_bounds__(256) void label_noise_kernel(const int32_t* y, const uint32_t* words, const int32_t* alt,
                                                          unsigned long long threshold, int n, int32_t* y_out, uint8_t* mask) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const bool hit = (unsigned long long)words[i] < threshold;
  y_out[i] = hit ? alt[i] : y[i];
  if (mask) mask[i] = hit ? 1 : 0;
}
void launch_label_noise(Ctx& ctx, const int32_t* y, const uint32_t* words, const int32_t* alt,
                        unsigned long long threshold, int n, int32_t* y_out, uint8_t* mask) {
  if (n <= 0) return;
  Launch l(ctx, BETTY_K_OTHER);
  label_noise_kernel<<<(n + 255) / 256, 256, 0, ctx.stream>>>(y, words, alt, threshold, n, y_out, mask);
}

}  // namespace betty
