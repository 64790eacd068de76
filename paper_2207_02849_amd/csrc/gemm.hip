// Grouped MFMA GEMM with fused epilogues for gfx950.
//
//   C (fp32 accumulators) = sum_p A_p * B_p^T  over one or two operand pairs, then an epilogue.
//
// Every dense contraction of the hypergradient path (forward, backward, and the forward-
// over-reverse passes of the Hessian-vector product; paper Sec. 3.2) has this shape because each
// operand is kept in the workspace with its reduction index contiguous ("K-major") and zero-
// padded to a multiple of 128 in both extents.  The two-pair form is the concatenated-K product
// of the R-op passes, e.g. Rz = Ra W + a V as [Ra | a] [W ; V].
//
// Launch = a batch of up to MAX_PROBLEMS independent problems plus optional bias-row jobs,
// flattened on blockIdx.x.  Problems with few output tiles are split along K *inside*
// the workgroup: KG wavefronts each take a contiguous range of k-tiles with their own
// LDS operand buffers, and their accumulators are summed through LDS in wavefront order, so the
// result is bit-reproducible and no inter-workgroup synchronisation exists (the smallest launches
// have a kernel of their own, gemm16_kernel).  (Splitting K across
// workgroups was measured first: the agent-scope fences it needs write back the L2 of every XCD
// and cost 10-80 us per launch on this chip.)
//
// Tiling: 4 wavefronts (2 x 2), or 8 (4 x 2) on the 128 x 64 tiles, own a BM x BN tile; a wavefront
// owns TM x TN MFMA blocks of 32 x 32.  K is consumed in tiles of NCH 16-byte chunks per row: global -> registers
// -> LDS with the next tile's global loads in flight during the multiplies.  LDS rows are padded
// by one chunk so the 16-byte fragment reads of 8 consecutive rows hit distinct banks.
//
// Fragments: lane l supplies row (l % 32) of the A block and of the B block; lanes 0-31 take the
// even chunks of the k-tile, lanes 32-63 the odd ones.  A chunk is 8 bf16 (one
// v_mfma_f32_32x32x16_bf16) or 4 floats (four v_mfma_f32_32x32x2_f32); A and B share the chunk
// assignment, so the order of k inside the product does not matter.  Register r of lane l holds
// C[8*(r/4) + 4*(l/32) + r%4][l%32]: four consecutive rows of one column per register quad, which
// is what the epilogues consume (one 4-element vector store into the transposed output).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace betty {

// ------------------------------------------------------------------------------------------
// epilogue helpers
// ------------------------------------------------------------------------------------------

// One 32x32 MFMA block as seen by one lane: 16 accumulators = rows rb + 8*(k/4) + k%4 (k = 0..15)
// of column col, with rb = block row + 4*(lane/32).  M, N = valid extent.
//
// The epilogue is split in two so that its memory latency hides behind the k loop: epi_prefetch
// (before the loop) issues every load the mode needs for the block's 16 elements into EpiRegs;
// epi_finish (after the loop) computes and stores.  Nothing the prefetch reads is written by the
// same launch before epi_finish of the same element.
// NR = 16: a whole block;  NR = 4: one register quad (four consecutive rows), rb already at its first row;
// NR = 1: a single element (gemm16_kernel).
template <int NR> struct EpiRegs { float a[NR], b[NR], c[NR], d[NR]; float colv; };

template <int NR> __device__ __forceinline__ int epi_row(int rb, int k) { return NR == 1 ? rb : NR == 16 ? rb + 8 * (k >> 2) + (k & 3) : rb + k; }

template <int NR>
__device__ __forceinline__ int epi_offset(int rb, int k, long long ld, int col) {
  return (int)((long long)epi_row<NR>(rb, k) * ld + col);   // layer slices are < 2^31 elements
}

template <int MODE, int NR>
__device__ __forceinline__ void epi_prefetch(const Epilogue& e, int M, int N, int rb, int col, EpiRegs<NR>& R) {
  if constexpr (MODE == EPI_RFWD_LAST_HESS) {
    // every lane of the block takes part in the row sums later: lanes outside the valid extent hold zeros
    const bool colok = col < N;
    if constexpr (NR > 1) R.colv = (colok && e.colvec) ? e.colvec[col] : 0.f;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int row = epi_row<NR>(rb, k);
      const bool ok = colok && row < M;
      R.a[k] = (ok && e.dphi) ? e.dphi[epi_offset<NR>(rb, k, e.ldf, col)] : 0.f;
      R.b[k] = ok ? e.e[row] : 0.f;
    }
    if constexpr (NR == 1) R.colv = (colok && e.colvec) ? e.colvec[col] : 0.f;      // (last: see below)
    return;
  }
  if (MODE == EPI_GRAM || (MODE == EPI_RBWD && e.mode == EPI_GRAM) || col >= N || rb >= M) return;
  const long long ldx = MODE >= EPI_WGRAD ? e.ldc : e.ldf;
  constexpr bool COLUMN = MODE == EPI_SAMPLE || MODE == EPI_FWD || MODE == EPI_FWD_LAST || MODE == EPI_RFWD || MODE == EPI_RFWD_LAST || MODE == EPI_FWD_PM;
  if constexpr (COLUMN && NR > 1) R.colv = e.colvec ? e.colvec[col] : 0.f;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const bool ok = epi_row<NR>(rb, k) < M;
    const int o = epi_offset<NR>(rb, k, ldx, col);
    if constexpr (MODE == EPI_FWD_PM) {
      R.a[k] = ok ? e.e[o] : 0.f;
      R.b[k] = e.Rz[0];
    } else if constexpr (MODE == EPI_BWD) {
      R.a[k] = ok ? e.dphi[o] : 0.f;
      R.b[k] = (ok && e.e_io) ? e.e_io[o] : 0.f;
    } else if constexpr (MODE == EPI_RFWD) {
      R.a[k] = ok ? e.dphi[o] : 0.f;
      R.b[k] = (ok && e.e) ? e.e[o] : 0.f;
    } else if constexpr (MODE == EPI_RFWD_LAST) {
      R.b[k] = (ok && e.e) ? e.e[o] : 0.f;
    } else if constexpr (MODE == EPI_SAMPLE) {
      R.a[k] = (ok && e.dphi) ? e.dphi[o] : 0.f;
      R.b[k] = (ok && e.e) ? e.e[o] : 0.f;
      R.c[k] = (ok && e.Rz) ? e.Rz[o] : 0.f;
    } else if constexpr (MODE == EPI_RBWD) {
      R.d[k] = (ok && e.e_io) ? e.e_io[o] : 0.f;
      R.a[k] = ok ? e.dphi[o] : 0.f;
      R.b[k] = (ok && e.e) ? e.e[o] : 0.f;
      R.c[k] = (ok && e.e) ? e.Rz[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD) {
      R.a[k] = (ok && e.lam) ? e.lam[o] : 0.f;
      R.b[k] = (ok && e.lam) ? e.x[o] : 0.f;
      R.c[k] = (ok && e.lam && e.p) ? e.p[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD_CG) {
      R.a[k] = ok ? e.x[o] : 0.f;
      R.c[k] = (ok && e.lam) ? e.lam[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD_NEUMANN) {
      R.a[k] = ok ? e.x[o] : 0.f;                         // s: the partial sum so far
      R.b[k] = ok ? e.v[o] : 0.f;                         // g: the vector the series is applied to
      R.c[k] = (ok && e.lam) ? e.lam[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD_NEUMANN_L2) {
      R.a[k] = ok ? e.p[o] : 0.f;                         // s
      R.b[k] = ok ? e.v[o] : 0.f;                         // g
      R.c[k] = ok ? e.lam[o] : 0.f;
      R.d[k] = ok ? e.x[o] : 0.f;                         // w
    } else if constexpr (MODE == EPI_WGRAD_FD || MODE == EPI_WGRAD_FD_LAST) {
      R.a[k] = ok ? e.v[o] : 0.f;
      R.b[k] = ok ? e.p[o] : 0.f;
      R.c[k] = (ok && e.lam) ? e.lam[o] : 0.f;
      if constexpr (MODE == EPI_WGRAD_FD_LAST) R.d[k] = (ok && e.x) ? e.x[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD_SCALED) {
      R.a[k] = ok ? e.x[o] : 0.f;
    } else if constexpr (MODE == EPI_WGRAD_SGD) {
      R.a[k] = ok ? e.v[o] : 0.f;
      R.b[k] = ok ? e.p[o] : 0.f;
      R.c[k] = (ok && e.lam) ? e.lam[o] : 0.f;
      R.d[k] = (ok && e.x) ? e.x[o] : 0.f;
    }
  }
  // (One element a lane: last.  The offset above is 64 bits wide on the way, with col's register and the one behind it, and was made to wait for
  // this value where it is loaded into that one.)
  if constexpr (COLUMN && NR == 1) R.colv = e.colvec ? e.colvec[col] : 0.f;
}

// the sums of a launch (Epilogue::partial): one number per finishing wavefront
template <int MODE> constexpr bool epi_sums() { return MODE == EPI_WGRAD || MODE == EPI_WGRAD_INIT || MODE == EPI_WGRAD_FD || MODE == EPI_WGRAD_SGD || MODE == EPI_WGRAD_CG; }
template <int MODE>
__device__ __forceinline__ void epi_store_sum(const Epilogue& e, int wave, double sum) {
  if constexpr (epi_sums<MODE>()) {
    if (!e.partial) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((threadIdx.x & 63) == 0) e.partial[4 * (size_t)blockIdx.x + wave] = sum;
  }
}

// a matrix over pairs of samples: fp32 as it is, bf16 as value and remainder (GemmArgs::split)
template <typename T, int NR>
__device__ __forceinline__ void epi_gram(const Epilogue& e, int M, int rb, int col, const float (&acc)[NR]) {
  T* o = (T*)e.out;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (epi_row<NR>(rb, k) >= M) continue;
    const float x = acc[k] + e.gamma;
    const long long at = (long long)epi_row<NR>(rb, k) * e.ld;
    if constexpr (sizeof(T) == 4) {
      o[at + col] = x;
    } else {
      const T hi = (T)x;
      o[at + (col >> 6) * 128 + (col & 63)] = hi;
      o[at + (col >> 6) * 128 + (col & 63) + 64] = (T)(x - (float)hi);
    }
  }
}

// operand-typed copies: row-major element by element, transposed as 4-element vectors; rows beyond M
// are written as zeros (they are padding of the transposed operand).  Either may be null.
template <typename T, int NR>
__device__ __forceinline__ void epi_copies(T* out, T* outT, int ld, int ldT, int M, int rb, int col, const bool (&ok)[NR], float (&val)[NR]) {
#pragma unroll
  for (int k = 0; k < NR; ++k)
    if (!ok[k]) val[k] = 0.f;
  if (out) {
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) store1<T>(out + (long long)epi_row<NR>(rb, k) * ld + col, val[k]);
  }
  if (outT) {
    T* o = outT + (long long)col * ldT + rb;
    if constexpr (NR == 1) {
      store1<T>(o, val[0]);
    } else {
#pragma unroll
      for (int q = 0; q < NR / 4; ++q) {
        const float quad[4] = {val[4 * q], val[4 * q + 1], val[4 * q + 2], val[4 * q + 3]};
        if (rb + 8 * q < M) store4<T>(o + 8 * q, quad);
      }
    }
  }
}

template <typename T, int MODE, int NR>
__device__ __forceinline__ void epi_finish(const Epilogue& e, int M, int N, int rb, int col,
                                           const float (&acc)[NR], const EpiRegs<NR>& R, float& sum) {
  float val[NR];
  if constexpr (MODE == EPI_RFWD_LAST_HESS) {
    // rows live across the 32 lanes of a half-wavefront (lane % 32 = column): butterfly sums
    const bool colok = col < N;
    float rz[NR], dot[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      rz[k] = colok ? acc[k] + R.colv : 0.f;
      dot[k] = R.a[k] * rz[k];
    }
    if (e.act == BETTY_LOSS_SOFTMAX_CE) {
#pragma unroll
      for (int o = NR == 1 ? 8 : 16; o > 0; o >>= 1)       // (16 lanes hold a row of a 16-tile)
#pragma unroll
        for (int k = 0; k < NR; ++k) dot[k] += __shfl_xor(dot[k], o, 64);
#pragma unroll
      for (int k = 0; k < NR; ++k) val[k] = R.b[k] * (R.a[k] * rz[k] - R.a[k] * dot[k]);
    } else {
#pragma unroll
      for (int k = 0; k < NR; ++k) val[k] = R.b[k] * 2.f * rz[k];
    }
  }
  if (col >= N || rb >= M) return;
  if (MODE == EPI_GRAM || (MODE == EPI_RBWD && e.mode == EPI_GRAM)) { epi_gram<T, NR>(e, M, rb, col, acc); return; }
  const long long ldx = MODE >= EPI_WGRAD ? e.ldc : e.ldf;
  bool ok[NR];
  int of[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    ok[k] = epi_row<NR>(rb, k) < M;
    of[k] = epi_offset<NR>(rb, k, ldx, col);
  }
  if constexpr (MODE == EPI_RFWD_LAST_HESS) {
    // val is set; fall through to the operand copies
  } else if constexpr (MODE == EPI_FWD_PM) {
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
      float* const dphi = sg ? e.d2_out : e.dphi_out;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        float d1, d2;
        const float t = R.b[k] * (e.alpha * (acc[k] + R.colv));
        act_eval(e.act, R.a[k] + (sg ? -t : t), val[k], d1, d2);
        if (ok[k]) dphi[of[k]] = d1;
      }
      epi_copies<T, NR>((T*)(sg ? e.out2 : e.out), (T*)(sg ? e.outT2 : e.outT), e.ld, e.ldT, M, rb, col, ok, val);
    }
    return;
  } else if constexpr (MODE == EPI_FWD) {
    float d1[NR], d2[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) act_eval(e.act, acc[k] + R.colv, val[k], d1[k], d2[k]);
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.dphi_out[of[k]] = d1[k];
    if (e.d2_out) {
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (ok[k]) e.d2_out[of[k]] = d2[k];
    }
    if constexpr (sizeof(T) == 4) {
      if (e.f0) {
#pragma unroll
        for (int k = 0; k < NR; ++k)
          if (ok[k]) e.f0[of[k]] = acc[k] + R.colv;
      }
    }
  } else if constexpr (MODE == EPI_SAMPLE) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const float sn = R.c[k] + (e.beta * R.b[k] - e.alpha * acc[k]) + R.colv;
      if (ok[k]) e.f0[of[k]] = sn;
      val[k] = R.a[k] * sn;
    }
  } else if constexpr (MODE == EPI_FWD_LAST) {
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.f0[of[k]] = acc[k] + R.colv;
    return;
  } else if constexpr (MODE == EPI_RFWD_LAST) {
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.f0[of[k]] = acc[k] + (R.colv + R.b[k]);
    return;
  } else if constexpr (MODE == EPI_BWD) {
    if (e.e_io) {
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (ok[k]) e.e_io[of[k]] = acc[k] * R.b[k];
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) val[k] = acc[k] * R.a[k];
  } else if constexpr (MODE == EPI_RFWD) {
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.f0[of[k]] = acc[k] + (R.colv + R.b[k]);
#pragma unroll
    for (int k = 0; k < NR; ++k) val[k] = R.a[k] * (acc[k] + (R.colv + R.b[k]));
  } else if constexpr (MODE == EPI_RBWD) {
#pragma unroll
    for (int k = 0; k < NR; ++k) val[k] = (acc[k] + R.d[k]) * R.a[k] + R.b[k] * R.c[k];
  } else if constexpr (MODE == EPI_WGRAD) {            // C = acc (+ 2 e^lam x)
    if (e.lam) {
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const float el = expf(R.a[k]), x = R.b[k] - R.c[k];
        if (ok[k]) { e.C[of[k]] = acc[k] + 2.f * el * x; sum += el * x * x; }
      }
    } else {
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (ok[k]) e.C[of[k]] = acc[k];
    }
    return;
  } else if constexpr (MODE == EPI_WGRAD_CG) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const float hx = e.lam ? acc[k] + 2.f * expf(R.c[k]) * R.a[k] : acc[k];
      if (ok[k]) { e.C[of[k]] = hx; sum += hx * R.a[k]; }
    }
    return;
  } else if constexpr (MODE == EPI_WGRAD_INIT) {       // v = acc (and p = acc if asked); operand copies
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      val[k] = acc[k];
      if (ok[k]) { e.v[of[k]] = acc[k]; if (e.p) e.p[of[k]] = acc[k]; sum += acc[k] * acc[k]; }
    }
  } else if constexpr (MODE == EPI_WGRAD_NEUMANN) {    // Hs = acc (+ 2 e^lam s); s <- g + s - alpha Hs
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      float hs = acc[k];
      if (e.lam) hs += 2.f * expf(R.c[k]) * R.a[k];
      val[k] = R.b[k] + (R.a[k] - e.alpha * hs);
    }
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.p[of[k]] = val[k];
  } else if constexpr (MODE == EPI_WGRAD_FD || MODE == EPI_WGRAD_FD_LAST) {
    const float eps = e.eps[0], scale = eps > 0.f ? 0.5f / eps : 0.f;      // v = 0 has the zero product
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const float el = e.lam ? 2.f * expf(R.c[k]) : 0.f;
      const float vn = R.a[k] - e.alpha * (acc[k] * scale + el * R.a[k]), pn = R.b[k] + vn;
      if (!ok[k]) continue;
      if constexpr (MODE == EPI_WGRAD_FD) {
        e.v[of[k]] = vn; e.p[of[k]] = pn;
        sum += e.sum_p ? pn * pn : vn * vn;
      } else {
        e.C[of[k]] = e.x ? fd_mixed_l2(R.c[k], R.d[k], e.alpha, pn) : el * (e.alpha * pn);
      }
    }
    return;
  } else if constexpr (MODE == EPI_WGRAD_SCALED) {
#pragma unroll
    for (int k = 0; k < NR; ++k)
      if (ok[k]) e.C[of[k]] = e.beta * R.a[k] - e.alpha * acc[k];
    return;
  } else if constexpr (MODE == EPI_WGRAD_SGD) {          // lower optimiser step: momentum SGD in place
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      float gk = acc[k] + e.gamma * R.b[k];
      if (e.lam) {                                                  // x: anchor of a proximal term
        const float el = expf(R.c[k]), x = R.b[k] - R.d[k];
        gk += 2.f * el * x;
        if (ok[k]) sum += el * x * x;
      }
      const float mk = e.beta * R.a[k] + gk;
      if (ok[k]) { e.v[of[k]] = mk; e.p[of[k]] = R.b[k] - e.alpha * mk; }
    }
    return;
  } else if constexpr (MODE == EPI_WGRAD_NEUMANN_L2) {  // final step: only d(lambda) leaves the kernel
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const float el = 2.f * expf(R.c[k]);
      const float sn = R.b[k] + (R.a[k] - e.alpha * (acc[k] + el * R.a[k]));
      if (ok[k]) e.C[of[k]] = -el * R.d[k] * (e.alpha * sn);
    }
    return;
  } else {
    return;
  }
  epi_copies<T, NR>((T*)e.out, (T*)e.outT, e.ld, e.ldT, M, rb, col, ok, val);
  if constexpr (MODE == EPI_FWD && sizeof(T) == 4)         // fp32 forward of a bf16 problem: the bf16 operand copies of the activation leave from here too
    epi_copies<__bf16, NR>((__bf16*)e.out2, (__bf16*)e.outT2, e.ld, e.ldT, M, rb, col, ok, val);
}

// ------------------------------------------------------------------------------------------
// the kernel
// ------------------------------------------------------------------------------------------

__device__ __forceinline__ float wave_sum_f(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// bias-shaped outputs: one wavefront per row of a K-major matrix, same update rules as the tiles
template <typename T, int MODE>
__device__ void bias_rows(const BiasJob& j, int row) {
  const int lane = threadIdx.x & 63;
  if (row >= j.rows) return;
  // 16 bytes per lane and access, two in flight; entries beyond k are zero padding of the operand
  constexpr int EPC = 16 / (int)sizeof(T);
  typedef __attribute__((__vector_size__(16))) T vecT;
  float acc = 0.f;
  for (const void* M = j.Mt; M; M = M == j.Mt ? j.Mt2 : nullptr) {
    const T* p = (const T*)M + (long long)row * j.ld + lane * EPC;
    for (int c = lane * EPC; c < j.k; c += 128 * EPC, p += 128 * EPC) {
      const vecT v0 = *(const vecT*)p;
      vecT v1{};
      if (c + 64 * EPC < j.k) v1 = *(const vecT*)(p + 64 * EPC);
#pragma unroll
      for (int i = 0; i < EPC; ++i) acc += (float)v0[i] + (float)v1[i];
    }
  }
  acc = wave_sum_f(acc);
  if (lane != 0) return;
  switch (MODE) {
    case EPI_WGRAD: {
      float g = acc, sum = 0.f;
      if (j.lam) {
        const float el = expf(j.lam[row]), x = j.x[row] - (j.p ? j.p[row] : 0.f);
        g += 2.f * el * x;
        sum = el * x * x;
      }
      j.C[row] = g;
      if (j.partial) j.partial[row] = sum;
      break;
    }
    case EPI_WGRAD_CG: {
      const float x = j.x[row], hx = j.lam ? acc + 2.f * expf(j.lam[row]) * x : acc;
      j.C[row] = hx;
      if (j.partial) j.partial[row] = hx * x;
      break;
    }
    case EPI_WGRAD_INIT:
      j.v[row] = acc;
      if (j.p) j.p[row] = acc;
      if (j.partial) j.partial[row] = acc * acc;
      break;
    case EPI_WGRAD_NEUMANN: {
      const float so = j.x[row];
      float hs = acc;
      if (j.lam) hs += 2.f * expf(j.lam[row]) * so;
      j.p[row] = j.v[row] + (so - j.alpha * hs);
      break;
    }
    case EPI_WGRAD_FD:
    case EPI_WGRAD_FD_LAST: {
      const float eps = j.eps[0], scale = eps > 0.f ? 0.5f / eps : 0.f;
      const float el = j.lam ? 2.f * expf(j.lam[row]) : 0.f, vo = j.v[row];
      const float vn = vo - j.alpha * (acc * scale + el * vo), pn = j.p[row] + vn;
      if (MODE == EPI_WGRAD_FD) {
        j.v[row] = vn; j.p[row] = pn;
        if (j.partial) j.partial[row] = j.sum_p ? pn * pn : vn * vn;
      } else {
        j.C[row] = j.x ? fd_mixed_l2(j.lam[row], j.x[row], j.alpha, pn) : el * (j.alpha * pn);
      }
      break;
    }
    case EPI_WGRAD_SCALED:
      j.C[row] = j.beta * j.x[row] - j.alpha * acc;
      break;
    case EPI_WGRAD_SGD: {
      const float wo = j.p[row];
      float gk = acc + j.gamma * wo, sum = 0.f;
      if (j.lam) {
        const float el = expf(j.lam[row]), x = wo - (j.x ? j.x[row] : 0.f);
        gk += 2.f * el * x;
        sum = el * x * x;
      }
      if (j.partial) j.partial[row] = sum;
      const float mk = j.beta * j.v[row] + gk;
      j.v[row] = mk;
      j.p[row] = wo - j.alpha * mk;
      break;
    }
    case EPI_WGRAD_NEUMANN_L2: {
      const float so = j.p[row], el = 2.f * expf(j.lam[row]);
      const float sn = j.v[row] + (so - j.alpha * (acc + el * so));
      j.C[row] = -el * j.x[row] * (j.alpha * sn);
      break;
    }
    default: break;
  }
}

template <int MODE> struct BatchOf {
  typedef std::conditional_t<(MODE >= EPI_WGRAD), WgradBatch,
                             std::conditional_t<(MODE == EPI_GRAM || MODE == EPI_SAMPLE), SampleBatch, ChainBatch>> type;
};

// (128-tiles are compiled for two resident workgroups per compute unit, so that one workgroup's
// epilogue traffic overlaps the other's k loop)
template <typename T, int BM, int BN, int NCH, int WPG, int KG, int MODE>
__global__ __launch_bounds__(64 * WPG * KG, (BM == 128 && KG == 1) ? 2 : 1) void gemm_fused_kernel(typename BatchOf<MODE>::type batch) {
  constexpr int GT = 64 * WPG;                     // threads of one K group
  constexpr int WM = WPG == 8 ? 4 : WPG == 4 ? 2 : 1, WN = WPG >= 4 ? 2 : 1;   // wavefronts of a group over the tile
  constexpr int ROW = NCH + 1;                     // LDS row pitch in 16-byte chunks
  constexpr int EPC = 16 / (int)sizeof(T);         // elements per chunk
  constexpr int KT = NCH * EPC;                    // elements per k-tile
  constexpr int TM = BM / (32 * WM), TN = BN / (32 * WN);   // 32x32 blocks per wavefront
  constexpr int LA = BM * NCH / GT, LB = BN * NCH / GT;
  // Two groups of four wavefronts (64-tiles): each takes half of K with LDS buffers of its own and all pass the same
  // barriers; the padding of the operands makes the number of k-tiles even.
  constexpr bool PAIR = KG == 2;
  static_assert(WPG == 1 ? KG >= 4 : WPG == 4 ? KG <= 2 : KG == 1, "K groups: one wavefront each, or two of four");
  static_assert(WPG == 1 || WPG == 4 || WPG == 8, "a K group is one wavefront, 2 x 2 or 4 x 2 wavefronts");
  static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0 && (BM * NCH) % GT == 0 && (BN * NCH) % GT == 0, "tile");
  extern __shared__ u32x4 smem[];

  // KG groups share the tile; group kg owns a contiguous range of k-tiles and its own LDS
  // operand buffers.  (Wavefront-uniform values are forced into scalar registers.)
  const int kg = __builtin_amdgcn_readfirstlane(threadIdx.x / GT);
  const int tid = threadIdx.x % GT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = WPG >= 4 ? wave >> 1 : 0, wn = WPG >= 4 ? wave & 1 : 0;
  // Unsplit launches keep two LDS operand buffers and alternate between them, so the stores of
  // one k-tile overlap the multiplication of the previous one and a k-tile costs one barrier.
  constexpr bool DB = KG == 1 || PAIR;
  constexpr int LBUF = (BM + BN) * ROW;            // one operand buffer, in chunks
  u32x4* sA = smem + kg * (PAIR ? 2 * LBUF : LBUF);
  u32x4* sB = sA + BM * ROW;
  // a one-wavefront group owns its LDS region alone: no workgroup barrier inside the k loop
#define BETTY_GROUP_SYNC() do { if constexpr (WPG == 1) __builtin_amdgcn_wave_barrier(); else __syncthreads(); } while (0)

  // ---- which job is this workgroup?
  int bid = blockIdx.x;
  if (bid >= batch.gemm_blocks) {
    bid -= batch.gemm_blocks;
    int j = 0;
    while (j + 1 < batch.n_bias && bid >= batch.bias_begin[j + 1]) ++j;
    bias_rows<T, MODE>(batch.bias[j], (bid - batch.bias_begin[j]) * (WPG * KG) + (threadIdx.x >> 6));
    return;
  }
  int pi = 0;
  while (pi + 1 < batch.n && bid >= batch.block_begin[pi + 1]) ++pi;
  const GemmArgs& g = batch.p[pi].g;
  const int tile = bid - batch.block_begin[pi];
  const int tiles_n = (g.N + BN - 1) / BN;
  int tm = tile / tiles_n, tn = tile % tiles_n;
  if (g.xgm > 0) {                                 // XCD-compact order (see GemmArgs)
    const int x = tile & 7, q = tile >> 3;
    const int rm = (g.M + BM - 1) / BM / g.xgm, rn = tiles_n / g.xgn;
    tm = (x / g.xgn) * rm + q / rn;
    tn = (x % g.xgn) * rn + q % rn;
  }
  const int m0 = tm * BM, n0 = tn * BN;

  const int sp = g.split;                          // (see GemmArgs::split)
  constexpr bool BSPLIT = MODE == EPI_WGRAD_SCALED;
  constexpr int KR = PAIR ? 2 : 1;                 // k-tiles come in whole multiples of the groups
  const int T0 = (g.K[0] + KR * KT - 1) / (KR * KT) * KR << sp, T1 = (g.K[1] + KR * KT - 1) / (KR * KT) * KR << sp, TT = T0 + T1;
  const int NI = (TT + KG - 1) / KG;               // iterations of every group (same barrier count)
  const int tb = kg * NI;
  const int te = tb + NI < TT ? tb + NI : TT;

  f32x16 acc[TM * TN];
#pragma unroll
  for (int i = 0; i < TM * TN; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  // epilogue inputs of this wavefront's blocks: requested now, consumed after the k loop.  Only
  // group 0 finishes the tile.  (With several blocks per wavefront the prefetch is kept for the
  // parameter-shaped modes, whose epilogue moves far more bytes than their k loop.)
  constexpr bool PREFETCH = TM * TN == 1 || (MODE >= EPI_WGRAD && BM == 64);
  // One-wavefront K groups: the tile is a single MFMA block, and once the groups' partial sums are
  // in LDS the first four wavefronts each finish one register quad of it (four consecutive rows
  // per lane), so the epilogue's arithmetic and stores run on four wavefronts instead of one.
  constexpr bool SPLIT_EPI = WPG == 1;
  const Epilogue& e = batch.p[pi].e;
  EpiRegs<16> pre[SPLIT_EPI || PAIR ? 1 : TM * TN];
  EpiRegs<4> pre4, pre4b;
  // A wavefront's loads return in the order issued, so a workgroup that requests its epilogue
  // inputs first starts its k loop only once they are there, and one that requests them last waits
  // for them after it: either way it streams and multiplies one after the other, and workgroups
  // that start together do so in step (the memory side idles while every k loop waits on operand
  // latency).  Parameter-shaped launches therefore alternate the two schedules between
  // neighbouring workgroups: one half streams while the other half multiplies (measured on the
  // Neumann weight-gradient launch of the 5M-parameter model: 28.3 -> 25.0 us).
  constexpr bool STAGGER = MODE >= EPI_WGRAD && BM == 64 && KG == 1;
  const bool early = !STAGGER || ((blockIdx.x >> 3) & 1) == 0;
  if constexpr (SPLIT_EPI) {
    if (kg < 4) epi_prefetch<MODE, 4>(e, g.M, g.N, m0 + 8 * kg + 4 * (lane >> 5), n0 + (lane & 31), pre4);
  } else if constexpr (PAIR) {
    // ... and of two groups' halves each group finishes two register quads of its four blocks
    epi_prefetch<MODE, 4>(e, g.M, g.N, m0 + wm * 32 + 16 * kg + 4 * (lane >> 5), n0 + wn * 32 + (lane & 31), pre4);
    epi_prefetch<MODE, 4>(e, g.M, g.N, m0 + wm * 32 + 16 * kg + 8 + 4 * (lane >> 5), n0 + wn * 32 + (lane & 31), pre4b);
  } else if constexpr (PREFETCH) {
    if (kg == 0 && early) {
#pragma unroll
      for (int ij = 0; ij < TM * TN; ++ij)
        epi_prefetch<MODE, 16>(e, g.M, g.N, m0 + wm * TM * 32 + (ij / TN) * 32 + 4 * (lane >> 5),
                               n0 + wn * TN * 32 + (ij % TN) * 32 + (lane & 31), pre[ij]);
    }
  }

  // Two register sets hold the global loads of the next two k-tiles, so two tiles' worth of
  // loads are in flight while a third is multiplied out of LDS (four sets in the long-loop form
  // of the unsplit activation-shaped launches, see below).
  constexpr bool LONG_LOOP = DB && MODE < EPI_WGRAD;
  u32x4 ra0[LA], rb0[LB], ra1[LA], rb1[LB];
  u32x4 ra2[LONG_LOOP ? LA : 1], rb2[LONG_LOOP ? LB : 1], ra3[LONG_LOOP ? LA : 1], rb3[LONG_LOOP ? LB : 1];
  // operand bases of both pairs are read from the kernel arguments once, not per k-tile
  const long long lda0 = g.lda[0], lda1 = g.lda[1], ldb0 = g.ldb[0], ldb1 = g.ldb[1];
  const T* const Abase0 = (const T*)g.A[0] + (long long)m0 * lda0 + (long long)(tid / NCH) * lda0 + (tid % NCH) * EPC;
  const T* const Abase1 = (const T*)g.A[1] + (long long)m0 * lda1 + (long long)(tid / NCH) * lda1 + (tid % NCH) * EPC;
  const T* const Bbase0 = (const T*)g.B[0] + (long long)n0 * ldb0 + (long long)(tid / NCH) * ldb0 + (tid % NCH) * EPC;
  const T* const Bbase1 = (const T*)g.B[1] + (long long)n0 * ldb1 + (long long)(tid / NCH) * ldb1 + (tid % NCH) * EPC;
#define BETTY_GLOAD(RA_, RB_, t_)                                                                    \
  {                                                                                                  \
    const bool second_ = (t_) >= T0;                                                                 \
    const int tt_ = second_ ? (t_) - T0 : (t_);                                                      \
    const T* Ab_ = (second_ ? Abase1 : Abase0) + (long long)(tt_ >> (BSPLIT && second_ ? sp : 0)) * KT; \
    const T* Bb_ = (second_ ? Bbase1 : Bbase0) + (long long)(tt_ >> (BSPLIT && second_ ? 0 : sp)) * KT; \
    const long long lda_ = (second_ ? lda1 : lda0) * (GT / NCH);                                    \
    const long long ldb_ = (second_ ? ldb1 : ldb0) * (GT / NCH);                                    \
    _Pragma("unroll") for (int i_ = 0; i_ < LA; ++i_) RA_[i_] = *(const u32x4*)(Ab_ + i_ * lda_);    \
    _Pragma("unroll") for (int i_ = 0; i_ < LB; ++i_) RB_[i_] = *(const u32x4*)(Bb_ + i_ * ldb_);    \
  }
  // one k-tile: registers -> LDS, refill the registers dist_ tiles ahead (always_, or if that tile
  // exists), multiply.  Every thread of the workgroup passes both barriers whether or not its group
  // still has a tile (t_ < te).
#define BETTY_STAGE(RA_, RB_, t_, first_, always_, dist_, buf_)                                      \
  {                                                                                                  \
    const bool live_ = DB || (t_) < te;                                                         \
    u32x4* const sA_ = sA + (DB ? (buf_) * LBUF : 0);                                                \
    u32x4* const sB_ = sB + (DB ? (buf_) * LBUF : 0);                                                \
    if (!DB && !(first_)) BETTY_GROUP_SYNC();                                                        \
    if (live_) {                                                                                     \
      _Pragma("unroll") for (int i_ = 0; i_ < LA; ++i_) {                                            \
        const int idx_ = tid + i_ * GT;                                                              \
        sA_[(idx_ / NCH) * ROW + idx_ % NCH] = RA_[i_];                                              \
      }                                                                                              \
      _Pragma("unroll") for (int i_ = 0; i_ < LB; ++i_) {                                            \
        const int idx_ = tid + i_ * GT;                                                              \
        sB_[(idx_ / NCH) * ROW + idx_ % NCH] = RB_[i_];                                              \
      }                                                                                              \
    }                                                                                                \
    BETTY_GROUP_SYNC();                                                                              \
    if ((always_) || (t_) + (dist_) < te) BETTY_GLOAD(RA_, RB_, (t_) + (dist_))                      \
    if (live_) {                                                                                     \
      _Pragma("unroll") for (int j_ = 0; j_ < NCH / 2; ++j_) {                                       \
        const int c_ = 2 * j_ + (lane >> 5);                                                         \
        u32x4 af_[TM], bf_[TN];                                                                      \
        _Pragma("unroll") for (int i_ = 0; i_ < TM; ++i_)                                            \
          af_[i_] = sA_[(wm * TM * 32 + i_ * 32 + (lane & 31)) * ROW + c_];                          \
        _Pragma("unroll") for (int i_ = 0; i_ < TN; ++i_)                                            \
          bf_[i_] = sB_[(wn * TN * 32 + i_ * 32 + (lane & 31)) * ROW + c_];                          \
        _Pragma("unroll") for (int i_ = 0; i_ < TM; ++i_)                                            \
          _Pragma("unroll") for (int jn_ = 0; jn_ < TN; ++jn_)                                       \
            MfmaChunk<T>::run(af_[i_], bf_[jn_], acc[i_ * TN + jn_]);                                \
      }                                                                                              \
    }                                                                                                \
  }

  const int n_full = te - tb;                       // tiles this group really has (<= NI)
  // Long-loop form, for unsplit activation-shaped launches with at least eight k-tiles.  What
  // counts for them is how many k-tiles are really in flight.  The compiler decides how long a
  // wavefront waits before it stores a register set to LDS from what it can prove about the loads
  // in flight, and where control flow merges it assumes the worst of the incoming paths: a refill
  // inside a branch, or a loop that can be entered with other loads in flight than its back edge
  // carries, makes every stage wait for all outstanding loads, i.e. for the tile requested one
  // stage ago, the full memory latency every other stage (512 x 4096 x 8192: 74 us).  Here the loop
  // is entered through straight-line code that leaves exactly the loop's own state, refills
  // unconditionally, and keeps four register sets, so a stage waits for the oldest set only while
  // three k-tiles stay in flight (66 us; 39 us for half the rows, which took 70 us before;
  // 8192 x 8192 x 4096 on 128-tiles 803 -> 695 us).
  bool done = false;
  if constexpr (LONG_LOOP) {
    if (n_full >= 8) {
      BETTY_GLOAD(ra0, rb0, tb)
      BETTY_GLOAD(ra1, rb1, tb + 1)
      BETTY_GLOAD(ra2, rb2, tb + 2)
      BETTY_GLOAD(ra3, rb3, tb + 3)
      int it = 0;
      for (; it + 7 < n_full; it += 4) {
        BETTY_STAGE(ra0, rb0, tb + it, false, true, 4, 0)
        BETTY_STAGE(ra1, rb1, tb + it + 1, false, true, 4, 1)
        BETTY_STAGE(ra2, rb2, tb + it + 2, false, true, 4, 0)
        BETTY_STAGE(ra3, rb3, tb + it + 3, false, true, 4, 1)
      }
      for (; it < n_full; it += 4) {                // the last four to seven tiles
        BETTY_STAGE(ra0, rb0, tb + it, false, false, 4, 0)
        if (it + 1 < n_full) BETTY_STAGE(ra1, rb1, tb + it + 1, false, false, 4, 1)
        if (it + 2 < n_full) BETTY_STAGE(ra2, rb2, tb + it + 2, false, false, 4, 0)
        if (it + 3 < n_full) BETTY_STAGE(ra3, rb3, tb + it + 3, false, false, 4, 1)
      }
      done = true;
    }
  }
  if (!done) {
    if (tb < te) BETTY_GLOAD(ra0, rb0, tb)
    if (tb + 1 < te) BETTY_GLOAD(ra1, rb1, tb + 1)
    // Unsplit launches (KG == 1) have long k loops: steady state while both refills of an iteration
    // stay inside the k-range, then a short tail.  K-split launches run a handful of tiles per
    // group; they keep the compact loop (less code to fetch for a kernel that lives a few us).
    int it = 0;
    if constexpr (DB) {
      if (n_full > 3) {                               // first pair peeled: no barrier before the first store
        BETTY_STAGE(ra0, rb0, tb, true, true, 2, 0)
        BETTY_STAGE(ra1, rb1, tb + 1, false, true, 2, 1)
        it = 2;
      }
      for (; it + 3 < n_full; it += 2) {
        BETTY_STAGE(ra0, rb0, tb + it, false, true, 2, 0)
        BETTY_STAGE(ra1, rb1, tb + it + 1, false, true, 2, 1)
      }
    }
    for (; it < NI; it += 2) {
      BETTY_STAGE(ra0, rb0, tb + it, it == 0, false, 2, 0)
      if (it + 1 < NI) BETTY_STAGE(ra1, rb1, tb + it + 1, false, false, 2, 1)
    }
  }
#undef BETTY_STAGE
#undef BETTY_GLOAD
#undef BETTY_GROUP_SYNC

  // ---- combine the K groups through LDS in group order (bit-reproducible); group 0 finishes
  if constexpr (SPLIT_EPI) {
    __syncthreads();                                // all groups are done with the operand tiles
    float* red = (float*)smem;
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(kg * 16 + r) * 64 + lane] = acc[0][r];
    __syncthreads();
    if (kg >= 4) return;
    float q4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) q4[r] = red[(4 * kg + r) * 64 + lane];
#pragma unroll 1
    for (int g2 = 1; g2 < KG; ++g2) {
#pragma unroll
      for (int r = 0; r < 4; ++r) q4[r] += red[((g2 * 16) + 4 * kg + r) * 64 + lane];
    }
    float sum = 0.f;
    epi_finish<T, MODE, 4>(e, g.M, g.N, m0 + 8 * kg + 4 * (lane >> 5), n0 + (lane & 31), q4, pre4, sum);
    epi_store_sum<MODE>(e, kg, sum);
    return;
  }

  if constexpr (PAIR) {
    __syncthreads();
    float* red = (float*)smem + (wave * 8) * 64 + lane;      // [group][wavefront][8 registers][lane]
#pragma unroll
    for (int r = 0; r < 8; ++r) red[(kg * 32 + r) * 64] = kg ? acc[0][r] : acc[0][8 + r];
    __syncthreads();
    float q4[4], q4b[4], sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      q4[r] = (kg ? acc[0][8 + r] : acc[0][r]) + red[((1 - kg) * 32 + r) * 64];
      q4b[r] = (kg ? acc[0][12 + r] : acc[0][4 + r]) + red[((1 - kg) * 32 + 4 + r) * 64];
    }
    epi_finish<T, MODE, 4>(e, g.M, g.N, m0 + wm * 32 + 16 * kg + 4 * (lane >> 5), n0 + wn * 32 + (lane & 31), q4, pre4, sum);
    epi_finish<T, MODE, 4>(e, g.M, g.N, m0 + wm * 32 + 16 * kg + 8 + 4 * (lane >> 5), n0 + wn * 32 + (lane & 31), q4b, pre4b, sum);
    return;
  }

  // ---- epilogue from registers, one MFMA block at a time
  float sum = 0.f;
#pragma unroll
  for (int ij = 0; ij < TM * TN; ++ij) {
    const int rb = m0 + wm * TM * 32 + (ij / TN) * 32 + 4 * (lane >> 5);
    const int col = n0 + wn * TN * 32 + (ij % TN) * 32 + (lane & 31);
    if (!PREFETCH || !early) epi_prefetch<MODE, 16>(e, g.M, g.N, rb, col, pre[ij]);
    float accf[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) accf[r] = acc[ij][r];
    epi_finish<T, MODE, 16>(e, g.M, g.N, rb, col, accf, pre[ij], sum);
  }
  epi_store_sum<MODE>(e, wave, sum);
}

// ------------------------------------------------------------------------------------------
// small launches: 16 x 16 tiles, operands in whole lines to LDS
// ------------------------------------------------------------------------------------------
//
// A launch whose output has few tiles is bound by dependent memory round trips (an empty kernel in a graph costs 1.75 us, one
// load-add-store per thread 1.85 us) and then by what the L1 of a compute unit takes in: 4 cycles a 128-byte line of a load,
// whether the load wants all of it or half.  16 rows x 64 bytes, a step of K in MFMA fragments, cost 65 cycles, 8 rows x 128 bytes 32.
// So a workgroup owns one 16 x 16 tile, its wavefronts split K, and each requests U pairs of steps (128 bytes of every operand row) at
// once, whole lines straight to LDS, and reads the fragments there: lane l holds row l % 16 and 16-byte chunk
// l / 16 of A and of B.  The chunks of row r stand in the order c ^ (r % 8), so that the rows spread over the banks.  Rows and
// pairs that nothing is multiplied with are not requested.  One round trip up to 32 pairs (fp32 K = 1024, bf16 2048), as many again for each
// further 32; 2 U to 8 U MFMA instructions, one pass through LDS
// (partial tiles summed in wavefront order, bit-reproducible), then one output element per thread.  Against steps
// straight into fragments: classifier 784-256-10, fp32, batch 128, K = 5 102.6 -> 95.9 us; conjugate gradient of 784-10, batch 512 159.5 -> 150.3;
// finite-difference step of 1023-509-251-10, batch 100 127.7 -> 121.2; a step of the series of n-48-48, batch 128, n = 1024, 2048, 4096:
// fp32 18.7 / 23.3 / 35.0 -> 16.5 / 19.7 / 27.5, bf16 16.0 / 18.4 / 20.7 -> 14.8 / 16.1 / 20.4.
// Short K goes straight into fragments, a step a wavefront (DIRECT): the way through LDS costs a launch more than the lines it saves.  Steps of eight
// layers, 32, 64, 128 wide, batch 256, by pairs and by steps: bf16 51.5 / 52.8 / 63.4 -> 46.3 / 49.4 / 60.7, fp32 54.0 / 56.7 -> 49.2 / 52.3
// (before there were pairs 48.9 / 52.0 / 61.8 and 52.1 / 54.4).  Of each, 1 to 2 us are the inputs of the epilogue that one wavefront's were
// waiting for (epi_prefetch), 2 us the partial tiles read four at a time.  The line: bf16 up to 10 steps (160-wide 65.3 us by steps, 66.1 by
// pairs; 192-wide 77.7 / 73.9 at batch 512), fp32 up to 12 (96-wide 68.0 / 70.1; 128-wide, 16 steps, 62.5 / 57.4 at batch 16).
// The two steps of a pair have a sum each, as two wavefronts would: fp32 products of K = 100 were 1.22 times as far off fp64 with one
// chain, calls of 90 GELU models 1.027 +- 0.004 times; with two, and MfmaSum16 in the narrow-output kernels, 0.92 times.  A call takes
// 0.2 % longer (0.5 at most).
constexpr int G16_PITCH = 17;                      // row pitch of a partial tile in LDS (floats)

// steps of K, 64 bytes of every operand row, and pairs of them (split: 64 elements, value and remainder)
__host__ __device__ __forceinline__ int small_steps(bool split, int K, int KS) { return split ? (K + 63) / 64 * 4 : (K + KS - 1) / KS; }
__host__ __device__ __forceinline__ int small_pairs(bool split, int K, int PK) { return split ? (K + 63) / 64 * 2 : (K + PK - 1) / PK; }

// DIRECT: a step a wavefront, straight into fragments
template <typename T, int U, bool DIRECT, int MODE>
__global__ __launch_bounds__(1024) void gemm16_kernel(typename BatchOf<MODE>::type batch) {
  constexpr int EPC = 16 / (int)sizeof(T), KS = 4 * EPC, PK = 2 * KS;      // elements per chunk, per step, per pair of steps
  extern __shared__ u32x4 smem[];
  const int t = threadIdx.x, lane = t & 63, kg = __builtin_amdgcn_readfirstlane(t >> 6), KG = blockDim.x >> 6;
  // A wavefront's partial tile, where its operands were: 16 wavefronts of one pair are 64 KB, and two workgroups fit a compute unit (beside the
  // operands 81 KB, and one: weight gradients of 660-73-73-34, bf16, batch 915 6.6 us, 5.1)
  constexpr int PART = DIRECT ? 16 * G16_PITCH : U * 1024;
  float* const part = (float*)smem;
  int bid = blockIdx.x;
  if constexpr (MODE >= EPI_WGRAD) {
    if (bid >= batch.gemm_blocks) {
      bid -= batch.gemm_blocks;
      int j = 0;
      while (j + 1 < batch.n_bias && bid >= batch.bias_begin[j + 1]) ++j;
      bias_rows<T, MODE>(batch.bias[j], (bid - batch.bias_begin[j]) * KG + kg);
      return;
    }
  }
  int pi = 0;
  while (pi + 1 < batch.n && bid >= batch.block_begin[pi + 1]) ++pi;
  const GemmArgs& g = batch.p[pi].g;
  const Epilogue& e = batch.p[pi].e;
  const int tile = bid - batch.block_begin[pi];
  const int tiles_n = (g.N + 15) >> 4;
  const int m0 = (tile / tiles_n) * 16, n0 = (tile % tiles_n) * 16;

  const int row = m0 + (t >> 4), col = n0 + (t & 15);      // the output element of threads 0..255
  EpiRegs<1> pre;
  if (t < 256) epi_prefetch<MODE, 1>(e, g.M, g.N, row, col, pre);

  const bool sp = g.split;
  const int fr = lane & 15;
  f32x4v acc = {0.f, 0.f, 0.f, 0.f};
  if constexpr (DIRECT) {
    const int S0 = small_steps(sp, g.K[0], KS), S = S0 + small_steps(sp, g.K[1], KS);
    const bool second = kg >= S0, bs = MODE == EPI_WGRAD_SCALED && second;
    const int qs = second ? kg - S0 : kg, qo = sp ? (qs >> 2 << 1) | (qs & 1) : qs;     // two steps of value, two of remainder
    const int ld_a = second ? g.lda[1] : g.lda[0], ld_b = second ? g.ldb[1] : g.ldb[0], fc = (lane >> 4) * EPC;
    u32x4 x = {}, y = {};
    if (kg < S) {
      if (m0 + fr < g.M) x = *(const u32x4*)((const T*)(second ? g.A[1] : g.A[0]) + (long long)(m0 + fr) * ld_a + (bs ? qo : qs) * KS + fc);
      if (n0 + fr < g.N) y = *(const u32x4*)((const T*)(second ? g.B[1] : g.B[0]) + (long long)(n0 + fr) * ld_b + (bs ? qs : qo) * KS + fc);
    }
    MfmaStep16<T>::run(x, y, acc);                             // (beyond the steps: zeros)
  } else {
    f32x4v odd = {0.f, 0.f, 0.f, 0.f};
    const int P0 = small_pairs(sp, g.K[0], PK), PT = P0 + small_pairs(sp, g.K[1], PK);
    const int per = (PT + KG - 1) / KG, p_begin = kg * per, p_end = min(PT, p_begin + per);
    // a lane's row and 16-byte chunk of a load of 8 rows x 128 bytes, chunks of a row in an order of its own (see below)
    const int lr = lane >> 3, lc = ((lane & 7) ^ lr) * EPC;
    const T* const A0 = (const T*)g.A[0] + (long long)(m0 + lr) * g.lda[0] + lc;
    const T* const B0 = (const T*)g.B[0] + (long long)(n0 + lr) * g.ldb[0] + lc;
    const T* const A1 = (const T*)g.A[1] + (long long)(m0 + lr) * g.lda[1] + lc;
    const T* const B1 = (const T*)g.B[1] + (long long)(n0 + lr) * g.ldb[1] + lc;
    const bool a_ok[2] = {m0 + lr < g.M, m0 + lr + 8 < g.M}, b_ok[2] = {n0 + lr < g.N, n0 + lr + 8 < g.N};
    char* const mine = (char*)smem + kg * U * 4096;            // this wavefront's operands: 16 rows of A, 16 of B a pair
    auto request = [&](const T* x, int ld, const bool (&ok)[2], char* to) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (ok[h])
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(x + (long long)(8 * h) * ld),
                                           (__attribute__((address_space(3))) void*)(to + 1024 * h), 16, 0, 0);
    };
    const int f0 = fr * 128 + (((lane >> 4) ^ fr) & 7) * 16, f1 = fr * 128 + ((((lane >> 4) + 4) ^ fr) & 7) * 16;
    for (int p = p_begin; p < p_end; p += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {                // (what nothing is multiplied with is not loaded: pairs beyond the range, rows beyond the output)
        const int q = p + u;
        if (q >= p_end) break;
        const bool second = q >= P0;
        const int qs = second ? q - P0 : q, qo = sp ? qs >> 1 : qs;          // a pair of value, one of remainder
        const bool bs = MODE == EPI_WGRAD_SCALED && second;
        request((second ? A1 : A0) + (long long)(bs ? qo : qs) * PK, second ? g.lda[1] : g.lda[0], a_ok, mine + u * 4096);
        request((second ? B1 : B0) + (long long)(bs ? qs : qo) * PK, second ? g.ldb[1] : g.ldb[0], b_ok, mine + u * 4096 + 2048);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (p + u >= p_end) break;
        const char* const x = mine + u * 4096;
        MfmaStep16<T>::run(*(const u32x4*)(x + f0), *(const u32x4*)(x + 2048 + f0), acc);
        MfmaStep16<T>::run(*(const u32x4*)(x + f1), *(const u32x4*)(x + 2048 + f1), odd);
      }
      if (p + U < p_end) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (read before they are overwritten)
    }
    acc += odd;
  }
  // register r of lane l is element [4 (l / 16) + r][l % 16]
#pragma unroll
  for (int r = 0; r < 4; ++r) part[kg * PART + (4 * (lane >> 4) + r) * G16_PITCH + fr] = acc[r];
  __syncthreads();
  if (t >= 256) return;
  float v[1] = {0.f};
  const float* const mine = part + (t >> 4) * G16_PITCH + (t & 15);
  for (int k = 0; k < KG; k += 4) {                  // (a multiple of four wavefronts, whose tiles' elements are read together)
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = mine[(k + i) * PART];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[0] += x[i];
  }
  float sum = 0.f;
  epi_finish<T, MODE, 1>(e, g.M, g.N, row, col, v, pre, sum);
  epi_store_sum<MODE>(e, kg, sum);
}

// ------------------------------------------------------------------------------------------
// weight-gradient launches of large layers (bf16 operands): 128 x 128 tiles, epilogue through LDS
// ------------------------------------------------------------------------------------------
//
// For a layer with millions of parameters the parameter-shaped epilogue (two or more fp32 vectors
// in, one out, two operand copies out) moves more bytes than the k loop, and with 64-tiles the
// operand panels cross the L2 -> L1 path twice as often.  This kernel keeps the k loop of
// gemm_fused_kernel at 128 x 128 but finishes the tile differently: the accumulators go to LDS once,
// then the tile is worked off in four passes of 32 rows in which a thread owns a 4 x 4 patch, so
// that every access to the flat fp32 vectors is a 16-byte access and eight neighbouring lanes
// cover a whole 128-byte line.  The inputs of pass p + 1 are requested before pass p is computed
// (those of pass 0 before the last two k-tiles are multiplied), and the transposed operand copy
// leaves through a small LDS staging tile as 16-byte rows.  Two workgroups fit a compute unit, so
// one streams its epilogue while the other multiplies.

// LAM: 0 = no diagonal term, 1 = with one, 2 = with one whose x is the distance to an anchor (mode WGRAD)
template <int MODE, int LAM> constexpr int wg_narr() {
  return MODE == EPI_WGRAD ? (LAM ? LAM + 1 : 0) : MODE == EPI_WGRAD_CG ? LAM + 1 : MODE == EPI_WGRAD_INIT ? 0 : MODE == EPI_WGRAD_NEUMANN ? (LAM ? 3 : 2)
       : MODE == EPI_WGRAD_SGD ? (LAM ? 4 : 2) : MODE == EPI_WGRAD_SCALED ? 1 : 4;
}
template <int MODE, int LAM> constexpr int wg_nreg() { return wg_narr<MODE, LAM>() > 0 ? wg_narr<MODE, LAM>() : 1; }

constexpr int WG_BT = 128;                 // tile extent
constexpr int WG_HP = WG_BT + 8;           // pitch of the fp32 accumulator tile in LDS (floats)
constexpr int WG_PASS = 32;                // rows per epilogue pass
constexpr int WG_TP = WG_PASS + 8;         // pitch of the transposed staging tile (elements)
constexpr size_t WG_LDS_OPERANDS = (size_t)2 * 2 * WG_BT * (GEMM_NCH + 1) * 16;
constexpr size_t WG_LDS_EPILOGUE = (size_t)WG_BT * WG_HP * 4 + (size_t)WG_BT * WG_TP * 2;
constexpr size_t WG_LDS = WG_LDS_OPERANDS > WG_LDS_EPILOGUE ? WG_LDS_OPERANDS : WG_LDS_EPILOGUE;

// what a workgroup needs of its problem's epilogue, read from the kernel arguments once
struct WgTile {
  const float* src[4];                     // fp32 inputs in the order the mode consumes them
  float* C; float* v; float* p;
  __bf16* out; __bf16* outT;
  long long ldc; int ld, ldT;
  int M, N, m0, n0;
  float alpha, beta, gamma;
  bool has_x;
};

// The flat fp32 vectors of a layer this large are streamed once per launch and come round again
// only after gigabytes of other traffic: their 16-byte accesses carry the non-temporal hint
// (121M-parameter model +3 %; the same hint on the operand copies, which the next launches read,
// loses 0.3 %).
// Rows and columns are clamped into the valid extent instead of being predicated, so the loads of
// all arrays of a patch are in flight together (a load inside control flow makes the compiler wait
// for the earlier ones first).  VEC: 16-byte accesses, whole patch inside the column extent.
template <bool VEC>
__device__ __forceinline__ void load_patch(const float* __restrict__ p, long long ld, int row0, int col0, int M, int N,
                                           float (&r)[4][4]) {
  if constexpr (VEC) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4v t = __builtin_nontemporal_load((const f32x4v*)(p + (long long)min(row0 + i, M - 1) * ld + col0));
      r[i][0] = t.x; r[i][1] = t.y; r[i][2] = t.z; r[i][3] = t.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) r[i][j] = p[(long long)min(row0 + i, M - 1) * ld + min(col0 + j, N - 1)];
  }
}

template <bool VEC>
__device__ __forceinline__ void store_patch(float* __restrict__ p, long long ld, int row0, int col0, int M, int N,
                                            const float (&r)[4][4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (row0 + i >= M) continue;
    float* q = p + (long long)(row0 + i) * ld + col0;
    if constexpr (VEC) {
      const f32x4v o4 = {r[i][0], r[i][1], r[i][2], r[i][3]};
      __builtin_nontemporal_store(o4, (f32x4v*)q);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (col0 + j < N) q[j] = r[i][j];
    }
  }
}

template <int MODE, int LAM, bool VEC>
__device__ __forceinline__ void wg_request(const WgTile& w, int pass, int pr, int pc, float (&in)[wg_nreg<MODE, LAM>()][4][4]) {
  constexpr int NARR = wg_narr<MODE, LAM>();
  const int row0 = w.m0 + WG_PASS * pass + 4 * pr, col0 = w.n0 + 4 * pc;
#pragma unroll
  for (int k = 0; k < NARR; ++k) load_patch<VEC>(w.src[k], w.ldc, row0, col0, w.M, w.N, in[k]);
}

// one pass of 32 rows: accumulators from LDS, the mode's update rule, stores.  Every thread of the
// workgroup calls it (it contains barriers when the transposed copy is asked for).
template <int MODE, int LAM, bool VEC>
__device__ __forceinline__ void wg_finish(const WgTile& w, int pass, int pr, int pc, int tid, const float* hs, __bf16* sT,
                                          const float (&in)[wg_nreg<MODE, LAM>()][4][4], float& sum) {
  constexpr int NR = wg_nreg<MODE, LAM>();
  // A row's terms are added before the next row's are made: the compiler would keep all 64 of the
  // tile and spill (gradients with a diagonal term, 10.4M parameters: 88 against 41 us).
  constexpr bool SUMS = MODE == EPI_WGRAD_INIT || MODE == EPI_WGRAD_CG || (LAM && (MODE == EPI_WGRAD || MODE == EPI_WGRAD_SGD));
  const int row0 = w.m0 + WG_PASS * pass + 4 * pr, col0 = w.n0 + 4 * pc;
  float acc[4][4], val[4][4], val2[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 h4 = *(const float4*)(hs + (WG_PASS * pass + 4 * pr + i) * WG_HP + 4 * pc);
    acc[i][0] = h4.x; acc[i][1] = h4.y; acc[i][2] = h4.z; acc[i][3] = h4.w;
  }
  const float (&I0)[4][4] = in[0];
  const float (&I1)[4][4] = in[NR > 1 ? 1 : 0];
  const float (&I2)[4][4] = in[NR > 2 ? 2 : 0];
  const float (&I3)[4][4] = in[NR > 3 ? 3 : 0];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = acc[i][j];
      const bool ok = row0 + i < w.M && (VEC || col0 + j < w.N);   // (what the sums count)
      if constexpr (MODE == EPI_WGRAD) {                   // I0 = lam, I1 = x, I2 = anchor
        val[i][j] = a;
        if constexpr (LAM) {
          const float el = expf(I0[i][j]), x = LAM == 2 ? I1[i][j] - I2[i][j] : I1[i][j];
          val[i][j] += 2.f * el * x;
          sum += ok ? el * x * x : 0.f;
        }
      } else if constexpr (MODE == EPI_WGRAD_CG) {         // I0 = x, I1 = lam
        val[i][j] = a;
        if constexpr (LAM) val[i][j] += 2.f * expf(I1[i][j]) * I0[i][j];
        sum += ok ? val[i][j] * I0[i][j] : 0.f;
      } else if constexpr (MODE == EPI_WGRAD_INIT) {
        val[i][j] = a;
        sum += ok ? a * a : 0.f;
      } else if constexpr (MODE == EPI_WGRAD_SCALED) {     // I0 = x
        val[i][j] = w.beta * I0[i][j] - w.alpha * a;
      } else if constexpr (MODE == EPI_WGRAD_NEUMANN) {    // I0 = s, I1 = g, I2 = lam
        float h = a;
        if constexpr (LAM) h += 2.f * expf(I2[i][j]) * I0[i][j];
        val[i][j] = I1[i][j] + (I0[i][j] - w.alpha * h);
      } else if constexpr (MODE == EPI_WGRAD_NEUMANN_L2) { // I0 = s, I1 = g, I2 = lam, I3 = w
        const float el = 2.f * expf(I2[i][j]);
        const float sn = I1[i][j] + (I0[i][j] - w.alpha * (a + el * I0[i][j]));
        val[i][j] = -el * I3[i][j] * (w.alpha * sn);
      } else {                                             // SGD: I0 = momentum, I1 = w, I2 = lam, I3 = anchor
        float gk = a + w.gamma * I1[i][j];
        if constexpr (LAM) {
          const float el = expf(I2[i][j]), x = I1[i][j] - (w.has_x ? I3[i][j] : 0.f);
          gk += 2.f * el * x;
          sum += ok ? el * x * x : 0.f;
        }
        const float mk = w.beta * I0[i][j] + gk;
        val[i][j] = mk;
        val2[i][j] = I1[i][j] - w.alpha * mk;
      }
    }
    if constexpr (SUMS) asm volatile("" : "+v"(sum));
  }
  if constexpr (MODE == EPI_WGRAD || MODE == EPI_WGRAD_CG || MODE == EPI_WGRAD_NEUMANN_L2 || MODE == EPI_WGRAD_SCALED) {
    store_patch<VEC>(w.C, w.ldc, row0, col0, w.M, w.N, val);
    return;
  } else if constexpr (MODE == EPI_WGRAD_SGD) {
    store_patch<VEC>(w.v, w.ldc, row0, col0, w.M, w.N, val);
    store_patch<VEC>(w.p, w.ldc, row0, col0, w.M, w.N, val2);
    return;
  } else {
    if constexpr (MODE == EPI_WGRAD_INIT) {
      store_patch<VEC>(w.v, w.ldc, row0, col0, w.M, w.N, val);
      if (w.p) store_patch<VEC>(w.p, w.ldc, row0, col0, w.M, w.N, val);
    } else {
      store_patch<VEC>(w.p, w.ldc, row0, col0, w.M, w.N, val);
    }
    // operand copies of the new vector: row-major [row][col] and transposed [col][row]; rows beyond
    // M inside a stored group are padding of the operand and are written as zeros
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (row0 + i >= w.M) {
#pragma unroll
        for (int j = 0; j < 4; ++j) val[i][j] = 0.f;
      }
    if (w.out) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (row0 + i >= w.M) continue;
        __bf16* o = w.out + (long long)(row0 + i) * w.ld + col0;
        if constexpr (VEC) {
          store4<__bf16>(o, val[i]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (col0 + j < w.N) o[j] = (__bf16)val[i][j];
        }
      }
    }
    if (w.outT) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float quad[4] = {val[0][j], val[1][j], val[2][j], val[3][j]};
        store4<__bf16>(sT + (4 * pc + j) * WG_TP + 4 * pr, quad);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = tid + 256 * u, c = q >> 2, k = q & 3;
        const int row = w.m0 + WG_PASS * pass + 8 * k;
        if (w.n0 + c < w.N && row < w.M)
          *(u32x4*)(w.outT + (long long)(w.n0 + c) * w.ldT + row) = *(const u32x4*)(sT + c * WG_TP + 8 * k);
      }
      __syncthreads();
    }
  }
}

// How many passes ahead the epilogue inputs are requested (the ring of register sets below holds
// one more).  Requesting the whole tile ahead (3, affordable with two input arrays) was measured
// slower than one pass ahead on the 121M-parameter model: 620 against 576 us per launch.  The final
// step of the series (four input arrays, once per hypergradient) requests each pass as it gets
// to it: a second register set would not fit beside the tile walk's state.  Nor would it where three
// or four arrays come with a sum (the anchored gradient, the SGD step of a diagonal cost).
template <int MODE, int LAM> constexpr int wg_depth() {
  return MODE == EPI_WGRAD_NEUMANN_L2 || (MODE == EPI_WGRAD && LAM == 2) || (MODE == EPI_WGRAD_SGD && LAM) ? 0 : 1;
}
constexpr int WG_NPASS = WG_BT / WG_PASS;

template <int MODE, int LAM, bool VEC>
__device__ __forceinline__ void wg_epilogue(const WgTile& w, int pr, int pc, int tid, const float* hs, __bf16* sT,
                                            float (&in)[wg_depth<MODE, LAM>() + 1][wg_nreg<MODE, LAM>()][4][4], float& sum) {
  constexpr int DEPTH = wg_depth<MODE, LAM>(), EARLY = DEPTH < 2 ? DEPTH : 2;
  // (with 16-byte accesses the first EARLY passes were requested inside the k loop)
#pragma unroll
  for (int q = VEC ? EARLY : 0; q < DEPTH; ++q) wg_request<MODE, LAM, VEC>(w, q, pr, pc, in[q]);
#pragma unroll
  for (int pass = 0; pass < WG_NPASS; ++pass) {
    if (pass + DEPTH < WG_NPASS) wg_request<MODE, LAM, VEC>(w, pass + DEPTH, pr, pc, in[(pass + DEPTH) % (DEPTH + 1)]);
    wg_finish<MODE, LAM, VEC>(w, pass, pr, pc, tid, hs, sT, in[pass % (DEPTH + 1)], sum);
  }
}

template <int MODE, int LAM>
__global__ __launch_bounds__(256, 2) void wgrad128_kernel(WgradBatch batch) {
  typedef __bf16 T;
  constexpr int BT = WG_BT, NCH = GEMM_NCH, ROW = NCH + 1, EPC = 8, KT = NCH * EPC, GT = 256;
  constexpr int LA = BT * NCH / GT;
  constexpr int LBUF = 2 * BT * ROW;
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // The first batch.walkers workgroups (two per compute unit) walk the tiles (tile = blockIdx.x,
  // then + walkers, ...) instead of one workgroup starting per tile, and where registers allow
  // request the first two k-tiles of their next tile before they finish the current one
  // (121M-parameter model: first weight-gradient launch 389 -> 370 us, Neumann launches 547 -> 536 us).
  // The bias rows follow in workgroups of their own.
  const int P = batch.walkers;
  if ((int)blockIdx.x >= P) {
    const int bid = blockIdx.x - P;
    int j = 0;
    while (j + 1 < batch.n_bias && bid >= batch.bias_begin[j + 1]) ++j;
    bias_rows<T, MODE>(batch.bias[j], (bid - batch.bias_begin[j]) * 4 + (threadIdx.x >> 6));
    return;
  }
  // patch of this thread inside an epilogue pass: eight lanes side by side cover 32 columns of four rows
  const int pc = 8 * wave + (lane & 7), pr = lane >> 3;

  // position and operands of a tile
  constexpr bool SPLIT = MODE == EPI_WGRAD_SCALED;      // (see GemmArgs::split)
  int pi, m0, n0, T0, TT, sp = 0;
  long long lda0, lda1, ldb0, ldb1;
  const T *Abase0, *Abase1, *Bbase0, *Bbase1;
#define BETTY_WG_LOCATE(tile_)                                                                       \
  {                                                                                                  \
    pi = 0;                                                                                          \
    while (pi + 1 < batch.n && (tile_) >= batch.block_begin[pi + 1]) ++pi;                           \
    const GemmArgs& g_ = batch.p[pi].g;                                                              \
    const int t_ = (tile_) - batch.block_begin[pi];                                                  \
    const int tiles_n_ = (g_.N + BT - 1) / BT;                                                       \
    int tm_ = t_ / tiles_n_, tn_ = t_ % tiles_n_;                                                    \
    if (g_.xgm > 0) {                                 /* XCD-compact order (see GemmArgs) */         \
      const int x_ = t_ & 7, q_ = t_ >> 3;                                                           \
      const int rm_ = (g_.M + BT - 1) / BT / g_.xgm, rn_ = tiles_n_ / g_.xgn;                        \
      tm_ = (x_ / g_.xgn) * rm_ + q_ / rn_;                                                          \
      tn_ = (x_ % g_.xgn) * rn_ + q_ % rn_;                                                          \
    }                                                                                                \
    m0 = tm_ * BT; n0 = tn_ * BT;                                                                    \
    if constexpr (SPLIT) sp = g_.split;                                                              \
    T0 = (g_.K[0] + 127) / 128 * 2 << sp; TT = T0 + ((g_.K[1] + 127) / 128 * 2 << sp);   /* an even number of k-tiles (operands are padded to 128) */ \
    lda0 = g_.lda[0]; lda1 = g_.lda[1]; ldb0 = g_.ldb[0]; ldb1 = g_.ldb[1];                          \
    Abase0 = (const T*)g_.A[0] + (long long)(m0 + tid / NCH) * lda0 + (tid % NCH) * EPC;             \
    Abase1 = (const T*)g_.A[1] + (long long)(m0 + tid / NCH) * lda1 + (tid % NCH) * EPC;             \
    Bbase0 = (const T*)g_.B[0] + (long long)(n0 + tid / NCH) * ldb0 + (tid % NCH) * EPC;             \
    Bbase1 = (const T*)g_.B[1] + (long long)(n0 + tid / NCH) * ldb1 + (tid % NCH) * EPC;             \
  }
  u32x4 ra0[LA], rb0[LA], ra1[LA], rb1[LA];
#define BETTY_WG_GLOAD(RA_, RB_, t_)                                                                 \
  {                                                                                                  \
    const bool second_ = (t_) >= T0;                                                                 \
    const int tt_ = second_ ? (t_) - T0 : (t_);                                                      \
    const T* Ab_ = (second_ ? Abase1 : Abase0) + (long long)(SPLIT && second_ ? tt_ >> sp : tt_) * KT;  \
    const T* Bb_ = (second_ ? Bbase1 : Bbase0) + (long long)(SPLIT && !second_ ? tt_ >> sp : tt_) * KT; \
    const long long lda_ = (second_ ? lda1 : lda0) * (GT / NCH);                                    \
    const long long ldb_ = (second_ ? ldb1 : ldb0) * (GT / NCH);                                    \
    _Pragma("unroll") for (int i_ = 0; i_ < LA; ++i_) RA_[i_] = *(const u32x4*)(Ab_ + i_ * lda_);    \
    _Pragma("unroll") for (int i_ = 0; i_ < LA; ++i_) RB_[i_] = *(const u32x4*)(Bb_ + i_ * ldb_);    \
  }
  // one k-tile: registers -> LDS buffer buf_, (refill the registers two tiles ahead), multiply.
  // Two buffers alternate, so a k-tile costs one barrier.
#define BETTY_WG_STAGE(RA_, RB_, t_, refill_, buf_)                                                  \
  {                                                                                                  \
    u32x4* const sA_ = smem + (buf_) * LBUF;                                                         \
    u32x4* const sB_ = sA_ + BT * ROW;                                                               \
    _Pragma("unroll") for (int i_ = 0; i_ < LA; ++i_) {                                              \
      const int idx_ = tid + i_ * GT;                                                                \
      sA_[(idx_ / NCH) * ROW + idx_ % NCH] = RA_[i_];                                                \
      sB_[(idx_ / NCH) * ROW + idx_ % NCH] = RB_[i_];                                                \
    }                                                                                                \
    __syncthreads();                                                                                 \
    if (refill_) BETTY_WG_GLOAD(RA_, RB_, (t_) + 2)                                                  \
    _Pragma("unroll") for (int j_ = 0; j_ < NCH / 2; ++j_) {                                         \
      const int c_ = 2 * j_ + (lane >> 5);                                                           \
      u32x4 af_[2], bf_[2];                                                                          \
      _Pragma("unroll") for (int i_ = 0; i_ < 2; ++i_) {                                             \
        af_[i_] = sA_[(wm * 64 + i_ * 32 + (lane & 31)) * ROW + c_];                                 \
        bf_[i_] = sB_[(wn * 64 + i_ * 32 + (lane & 31)) * ROW + c_];                                 \
      }                                                                                              \
      _Pragma("unroll") for (int i_ = 0; i_ < 2; ++i_)                                               \
        _Pragma("unroll") for (int jn_ = 0; jn_ < 2; ++jn_)                                          \
          MfmaChunk<T>::run(af_[i_], bf_[jn_], acc[i_ * 2 + jn_]);                                   \
    }                                                                                                \
  }

  float* const hs = (float*)smem;
  __bf16* const sT = (__bf16*)(hs + BT * WG_HP);
  int tile = blockIdx.x;
  float sum = 0.f;
  double tiles_sum = 0.0;
  BETTY_WG_LOCATE(tile)
  BETTY_WG_GLOAD(ra0, rb0, 0)
  BETTY_WG_GLOAD(ra1, rb1, 1)
  for (;;) {
    // here the first two k-tiles of `tile` are in flight and pi, m0, n0, TT, the bases describe it
    const Epilogue& e = batch.p[pi].e;
    WgTile w;
    w.C = e.C; w.v = e.v; w.p = e.p; w.out = (T*)e.out; w.outT = (T*)e.outT;
    w.ldc = e.ldc; w.ld = e.ld; w.ldT = e.ldT;
    w.M = batch.p[pi].g.M; w.N = batch.p[pi].g.N; w.m0 = m0; w.n0 = n0;
    w.alpha = e.alpha; w.beta = e.beta; w.gamma = e.gamma;
    w.has_x = e.x != nullptr;
    if constexpr (MODE == EPI_WGRAD) { w.src[0] = e.lam; w.src[1] = e.x; w.src[2] = e.p; w.src[3] = e.lam; }
    else if constexpr (MODE == EPI_WGRAD_CG) { w.src[0] = e.x; w.src[1] = e.lam; w.src[2] = w.src[3] = e.x; }
    else if constexpr (MODE == EPI_WGRAD_NEUMANN) { w.src[0] = e.x; w.src[1] = e.v; w.src[2] = e.lam; w.src[3] = e.x; }
    else if constexpr (MODE == EPI_WGRAD_NEUMANN_L2) { w.src[0] = e.p; w.src[1] = e.v; w.src[2] = e.lam; w.src[3] = e.x; }
    else if constexpr (MODE == EPI_WGRAD_SCALED) { w.src[0] = e.x; w.src[1] = w.src[2] = w.src[3] = e.x; }
    else if constexpr (MODE == EPI_WGRAD_SGD) { w.src[0] = e.v; w.src[1] = e.p; w.src[2] = e.lam; w.src[3] = e.x ? e.x : e.p; }
    else { w.src[0] = w.src[1] = w.src[2] = w.src[3] = nullptr; }
    // 16-byte accesses need every flat vector of the tile aligned and the tile inside the columns
    unsigned long long bits = (unsigned long long)w.C | (unsigned long long)w.v | (unsigned long long)w.p;
#pragma unroll
    for (int k = 0; k < wg_narr<MODE, LAM>(); ++k) bits |= (unsigned long long)w.src[k];
    const bool vec = (bits & 15) == 0 && (w.ldc & 3) == 0 && n0 + BT <= w.N;

    f32x16 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    int it = 0;
    for (; it + 2 < TT; it += 2) {
      BETTY_WG_STAGE(ra0, rb0, it, true, 0)
      BETTY_WG_STAGE(ra1, rb1, it + 1, true, 1)
    }
    // every operand load is issued: request the inputs of the first epilogue pass behind them
    float in[wg_depth<MODE, LAM>() + 1][wg_nreg<MODE, LAM>()][4][4];
    if (vec) {
#pragma unroll
      for (int q = 0; q < (wg_depth<MODE, LAM>() < 2 ? wg_depth<MODE, LAM>() : 2); ++q) wg_request<MODE, LAM, true>(w, q, pr, pc, in[q]);
    }
    BETTY_WG_STAGE(ra0, rb0, it, false, 0)
    BETTY_WG_STAGE(ra1, rb1, it + 1, false, 1)

    // accumulators -> LDS (the operand buffers are dead): register r of lane l of block (i, j) is
    // element [64 wm + 32 i + 8 (r / 4) + 4 (l / 32) + r % 4][64 wn + 32 j + l % 32]
    __syncthreads();
#pragma unroll
    for (int ij = 0; ij < 4; ++ij)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        hs[(wm * 64 + (ij >> 1) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * WG_HP + wn * 64 + (ij & 1) * 32 + (lane & 31)] = acc[ij][r];
    __syncthreads();

    // the next tile's first two k-tiles, requested ahead of this tile's epilogue (after the last
    // tile the same tile once more: no branch around the loads, see gemm_fused_kernel's long loop)
    // (only in the modes whose epilogue reads nothing: with epilogue inputs in flight as well the
    // request ahead gains nothing measurable, and with three or four input arrays there are no
    // registers for it)
    constexpr bool AHEAD = wg_narr<MODE, LAM>() == 0;
    const int next = tile + P;
    const bool more = next < batch.gemm_blocks;
    if constexpr (AHEAD) {
      BETTY_WG_LOCATE(more ? next : tile)
      BETTY_WG_GLOAD(ra0, rb0, 0)
      BETTY_WG_GLOAD(ra1, rb1, 1)
    }
    if (vec) wg_epilogue<MODE, LAM, true>(w, pr, pc, tid, hs, sT, in, sum);
    else wg_epilogue<MODE, LAM, false>(w, pr, pc, tid, hs, sT, in, sum);
    if constexpr (epi_sums<MODE>()) { tiles_sum += sum; sum = 0.f; }
    if (!more) { epi_store_sum<MODE>(e, wave, tiles_sum); break; }
    __syncthreads();                                // the next k loop writes where this epilogue read
    tile = next;
    if constexpr (!AHEAD) {
      BETTY_WG_LOCATE(tile)
      BETTY_WG_GLOAD(ra0, rb0, 0)
      BETTY_WG_GLOAD(ra1, rb1, 1)
    }
  }
#undef BETTY_WG_STAGE
#undef BETTY_WG_GLOAD
#undef BETTY_WG_LOCATE
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------

// the by-value argument block of a launch, cut to its kind
template <int MODE>
static typename BatchOf<MODE>::type kernel_args(const GemmBatch& b) {
  typename BatchOf<MODE>::type c;
  c.n = b.n; c.n_bias = b.n_bias; c.gemm_blocks = b.gemm_blocks; c.walkers = b.walkers;
  for (int i = 0; i <= b.n; ++i) c.block_begin[i] = b.block_begin[i];
  for (int i = 0; i < b.n; ++i) c.p[i] = b.p[i];
  if constexpr (MODE >= EPI_WGRAD) {
    for (int i = 0; i <= b.n_bias; ++i) c.bias_begin[i] = b.bias_begin[i];
    for (int i = 0; i < b.n_bias; ++i) c.bias[i] = b.bias[i];
  }
  return c;
}
static int max_problems(int mode) { return mode >= EPI_WGRAD ? MAX_PROBLEMS : mode >= EPI_GRAM ? MAX_SAMPLE_PROBLEMS : MAX_CHAIN_PROBLEMS; }

template <typename T, int BT, int WPG, int KG>
constexpr size_t lds_bytes() {
  constexpr size_t operands = (size_t)(KG <= 2 ? 2 * KG : KG) * 2 * BT * (GEMM_NCH + 1) * 16;
  constexpr size_t reduce = WPG == 1 ? (size_t)KG * BT * BT * 4 : 0;
  return operands > reduce ? operands : reduce;
}

template <typename T, int BT, int WPG, int KG, int MODE>
static void launch_one(int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  constexpr size_t lds = lds_bytes<T, BT, WPG, KG>();
  if constexpr (lds > 48 * 1024) {
    static PerDevice allowed;
    if (const hipError_t e = allow_lds(allowed, (const void*)gemm_fused_kernel<T, BT, BT, GEMM_NCH, WPG, KG, MODE>, lds); e != hipSuccess) { err = e; return; }
  }
  gemm_fused_kernel<T, BT, BT, GEMM_NCH, WPG, KG, MODE><<<total, 64 * WPG * KG, lds, st>>>(kernel_args<MODE>(b));
}

// 128 x 64 tiles, unsplit, eight wavefronts with one MFMA block each (a launch of these tiles puts
// one workgroup on a compute unit, and two wavefronts per SIMD hide each other's barrier and LDS
// waits: 121M-parameter model +2.3 % over four wavefronts of two blocks): the activation-shaped
// products of a grid that would otherwise leave one to four 64-tiles per compute unit
template <typename T, int MODE>
static void launch_rect(int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  constexpr size_t lds = (size_t)2 * (128 + 64) * (GEMM_NCH + 1) * 16;
  static PerDevice allowed;
  if (const hipError_t e = allow_lds(allowed, (const void*)gemm_fused_kernel<T, 128, 64, GEMM_NCH, 8, 1, MODE>, lds); e != hipSuccess) { err = e; return; }
  gemm_fused_kernel<T, 128, 64, GEMM_NCH, 8, 1, MODE><<<total, 512, lds, st>>>(kernel_args<MODE>(b));
}

template <typename T>
static void launch_rect_mode(int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  switch (mode) {
#define BETTY_CASE_R(M_) case M_: launch_rect<T, M_>(total, st, b, err); break;
    BETTY_CASE_R(EPI_FWD) BETTY_CASE_R(EPI_FWD_LAST) BETTY_CASE_R(EPI_BWD) BETTY_CASE_R(EPI_RFWD)
    BETTY_CASE_R(EPI_RFWD_LAST) BETTY_CASE_R(EPI_RBWD) BETTY_CASE_R(EPI_RFWD_LAST_HESS) BETTY_CASE_R(EPI_GRAM) BETTY_CASE_R(EPI_SAMPLE)
    case EPI_FWD_PM:
      if constexpr (sizeof(T) == 4) launch_rect<T, EPI_FWD_PM>(total, st, b, err);
      else err = hipErrorInvalidValue;
      break;
#undef BETTY_CASE_R
    default: err = hipErrorInvalidValue; break;
  }
}

template <typename T, int BT, int WPG, int KG>
static void launch_chain_mode(int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  switch (mode) {
#define BETTY_CASE(M_) case M_: launch_one<T, BT, WPG, KG, M_>(total, st, b, err); break;
    BETTY_CASE(EPI_FWD) BETTY_CASE(EPI_FWD_LAST) BETTY_CASE(EPI_BWD) BETTY_CASE(EPI_RFWD)
    BETTY_CASE(EPI_RFWD_LAST) BETTY_CASE(EPI_RBWD) BETTY_CASE(EPI_RFWD_LAST_HESS) BETTY_CASE(EPI_GRAM) BETTY_CASE(EPI_SAMPLE)
    case EPI_FWD_PM:
      if constexpr (sizeof(T) == 4 && BT < 128) launch_one<T, BT, WPG, KG, EPI_FWD_PM>(total, st, b, err);
      else err = hipErrorInvalidValue;
      break;
    default: err = hipErrorInvalidValue; break;
  }
}

template <typename T, int BT, int WPG, int KG>
static void launch_wgrad_mode(int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  switch (mode) {
#define BETTY_CASE_W(M_) case M_: launch_one<T, BT, WPG, KG, M_>(total, st, b, err); break;
    BETTY_CASE_W(EPI_WGRAD) BETTY_CASE_W(EPI_WGRAD_INIT) BETTY_CASE_W(EPI_WGRAD_NEUMANN)
    BETTY_CASE_W(EPI_WGRAD_NEUMANN_L2) BETTY_CASE_W(EPI_WGRAD_SGD) BETTY_CASE_W(EPI_WGRAD_SCALED)
    BETTY_CASE_W(EPI_WGRAD_FD) BETTY_CASE_W(EPI_WGRAD_FD_LAST) BETTY_CASE_W(EPI_WGRAD_CG)
#undef BETTY_CASE_W
    default: err = hipErrorInvalidValue; break;
  }
}
#undef BETTY_CASE

template <int MODE, int LAM>
static void launch_wgrad128_one(int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  static PerDevice allowed;
  if (const hipError_t e = allow_lds(allowed, (const void*)wgrad128_kernel<MODE, LAM>, WG_LDS); e != hipSuccess) { err = e; return; }
  wgrad128_kernel<MODE, LAM><<<total - b.gemm_blocks + b.walkers, 256, WG_LDS, st>>>(kernel_args<MODE>(b));
}

// bf16 weight-gradient launches on 128-tiles; the L2-decay term (lam) is the same for every problem of a batch
static void launch_wgrad128(int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  const bool lam = b.p[0].e.lam != nullptr;
  switch (mode) {
#define BETTY_CASE_W(M_) case M_: if (lam) launch_wgrad128_one<M_, 1>(total, st, b, err); else launch_wgrad128_one<M_, 0>(total, st, b, err); break;
    case EPI_WGRAD:
      if (lam && b.p[0].e.p) launch_wgrad128_one<EPI_WGRAD, 2>(total, st, b, err);
      else if (lam) launch_wgrad128_one<EPI_WGRAD, 1>(total, st, b, err);
      else launch_wgrad128_one<EPI_WGRAD, 0>(total, st, b, err);
      break;
    BETTY_CASE_W(EPI_WGRAD_NEUMANN) BETTY_CASE_W(EPI_WGRAD_SGD) BETTY_CASE_W(EPI_WGRAD_CG)
#undef BETTY_CASE_W
    case EPI_WGRAD_INIT: launch_wgrad128_one<EPI_WGRAD_INIT, 0>(total, st, b, err); break;
    case EPI_WGRAD_SCALED: launch_wgrad128_one<EPI_WGRAD_SCALED, 0>(total, st, b, err); break;
    case EPI_WGRAD_NEUMANN_L2: launch_wgrad128_one<EPI_WGRAD_NEUMANN_L2, 1>(total, st, b, err); break;
    default: err = hipErrorInvalidValue; break;
  }
}

// gemm16_kernel: wavefronts (kg), pairs of steps per wavefront and round (u; 0: a step a wavefront)
struct Small { int u, kg; };
template <typename T>
static Small small_shape(const GemmBatch& b) {
  constexpr int KS = 64 / (int)sizeof(T), DIRECT = sizeof(T) == 2 ? 10 : 12;
  int S = 1, P = 1;
  for (int i = 0; i < b.n; ++i) {
    const GemmArgs& g = b.p[i].g;
    S = std::max(S, small_steps(g.split, g.K[0], KS) + small_steps(g.split, g.K[1], KS));
    P = std::max(P, small_pairs(g.split, g.K[0], 2 * KS) + small_pairs(g.split, g.K[1], 2 * KS));
  }
  if (S <= DIRECT) return Small{0, (S + 3) / 4 * 4};
  const int u = P > 16 ? 2 : 1, per = std::max(u, (P + 15) / 16);
  return Small{u, ((P + per - 1) / per + 3) / 4 * 4};
}

template <typename T, int U, int MODE>
static void launch_small_one(int total, int kg, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  static PerDevice allowed;
  if (const hipError_t e = allow_lds(allowed, (const void*)gemm16_kernel<T, U, false, MODE>, 16 * U * 4096); e != hipSuccess) { err = e; return; }
  gemm16_kernel<T, U, false, MODE><<<total, 64 * kg, (size_t)kg * U * 4096, st>>>(kernel_args<MODE>(b));
}
template <typename T, int MODE>
static void launch_small(int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  const Small sh = small_shape<T>(b);
  if (sh.u == 0) gemm16_kernel<T, 1, true, MODE><<<total, 64 * sh.kg, (size_t)sh.kg * 16 * G16_PITCH * 4, st>>>(kernel_args<MODE>(b));
  else if (sh.u == 1) launch_small_one<T, 1, MODE>(total, sh.kg, st, b, err);
  else launch_small_one<T, 2, MODE>(total, sh.kg, st, b, err);
}

template <typename T>
static void launch_small_mode(int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  switch (mode) {
#define BETTY_CASE_S(M_) case M_: launch_small<T, M_>(total, st, b, err); break;
    BETTY_CASE_S(EPI_FWD) BETTY_CASE_S(EPI_FWD_LAST) BETTY_CASE_S(EPI_BWD) BETTY_CASE_S(EPI_RFWD)
    BETTY_CASE_S(EPI_RFWD_LAST) BETTY_CASE_S(EPI_RBWD) BETTY_CASE_S(EPI_RFWD_LAST_HESS) BETTY_CASE_S(EPI_GRAM) BETTY_CASE_S(EPI_SAMPLE)
    case EPI_FWD_PM:
      if constexpr (sizeof(T) == 4) launch_small<T, EPI_FWD_PM>(total, st, b, err);
      else err = hipErrorInvalidValue;
      break;
    BETTY_CASE_S(EPI_WGRAD) BETTY_CASE_S(EPI_WGRAD_INIT) BETTY_CASE_S(EPI_WGRAD_NEUMANN)
    BETTY_CASE_S(EPI_WGRAD_NEUMANN_L2) BETTY_CASE_S(EPI_WGRAD_SGD) BETTY_CASE_S(EPI_WGRAD_SCALED)
    BETTY_CASE_S(EPI_WGRAD_FD) BETTY_CASE_S(EPI_WGRAD_FD_LAST) BETTY_CASE_S(EPI_WGRAD_CG)
#undef BETTY_CASE_S
    default: err = hipErrorInvalidValue; break;
  }
}

template <typename T>
static void launch_elem(int cfg, int mode, int total, hipStream_t st, const GemmBatch& b, hipError_t& err) {
  if (b.n > max_problems(mode)) { err = hipErrorInvalidValue; return; }
  if (cfg == GEMM_16) { launch_small_mode<T>(mode, total, st, b, err); return; }
  if (mode >= EPI_WGRAD) {
    if (cfg == GEMM_128x1 && sizeof(T) == 2) launch_wgrad128(mode, total, st, b, err);
    else if (cfg == GEMM_128x1) launch_wgrad_mode<T, 128, 4, 1>(mode, total, st, b, err);
    else if (cfg == GEMM_64x1) launch_wgrad_mode<T, 64, 4, 1>(mode, total, st, b, err);
    else if (cfg == GEMM_32x8) launch_wgrad_mode<T, 32, 1, 8>(mode, total, st, b, err);
    else err = hipErrorInvalidValue;
    return;
  }
  switch (cfg) {
    case GEMM_128x1: launch_chain_mode<T, 128, 4, 1>(mode, total, st, b, err); break;
    case GEMM_64x1: launch_chain_mode<T, 64, 4, 1>(mode, total, st, b, err); break;
    case GEMM_32x8: launch_chain_mode<T, 32, 1, 8>(mode, total, st, b, err); break;
    case GEMM_32x4:                                  // first-order passes of optimiser steps only (plan_chain)
      if (mode == EPI_FWD) launch_one<T, 32, 1, 4, EPI_FWD>(total, st, b, err);
      else if (mode == EPI_FWD_LAST) launch_one<T, 32, 1, 4, EPI_FWD_LAST>(total, st, b, err);
      else if (mode == EPI_BWD) launch_one<T, 32, 1, 4, EPI_BWD>(total, st, b, err);
      else err = hipErrorInvalidValue;
      break;
    case GEMM_64x2: launch_chain_mode<T, 64, 4, 2>(mode, total, st, b, err); break;
    case GEMM_128x64: launch_rect_mode<T>(mode, total, st, b, err); break;
    default: err = hipErrorInvalidValue; break;
  }
}

// compute units of the current device (asked once; every device of a node is the same part)
static int resident_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else { (void)hipGetLastError(); cus = 256; }
  }
  return cus;
}

int gemm_cfg_tile(int cfg) { return cfg == GEMM_128x1 ? 128 : (cfg == GEMM_32x8 || cfg == GEMM_32x4) ? 32 : cfg == GEMM_16 ? 16 : 64; }   // (columns, for 128x64)
static int gemm_cfg_tile_rows(int cfg) { return cfg == GEMM_128x64 ? 128 : gemm_cfg_tile(cfg); }
static int gemm_cfg_waves(int cfg) { return cfg == GEMM_32x8 ? 8 : 4; }

int launch_gemm_batch(Ctx& ctx, Elem elem, int cfg, GemmBatch& b, double flops, double bytes, double* partial) {
  const int bt = gemm_cfg_tile(cfg);
  const int rows_per_block = cfg != GEMM_16 ? gemm_cfg_waves(cfg)
                           : (elem == ELEM_BF16 ? small_shape<__bf16>(b) : small_shape<float>(b)).kg;
  int blocks = 0;
  for (int i = 0; i < b.n; ++i) {
    b.block_begin[i] = blocks;
    const int br = gemm_cfg_tile_rows(cfg);
    blocks += ((b.p[i].g.M + br - 1) / br) * ((b.p[i].g.N + bt - 1) / bt);
  }
  b.block_begin[b.n] = blocks;
  b.gemm_blocks = blocks;
  b.walkers = blocks < 2 * resident_cus() ? blocks : 2 * resident_cus();
  int bias_blocks = 0;
  for (int i = 0; i < b.n_bias; ++i) {
    b.bias_begin[i] = bias_blocks;
    bias_blocks += (b.bias[i].rows + rows_per_block - 1) / rows_per_block;
  }
  b.bias_begin[b.n_bias] = bias_blocks;
  const int total = blocks + bias_blocks;
  if (total <= 0) return 0;
  int n_partial = 0;
  if (partial) {
    n_partial = 4 * (elem == ELEM_BF16 && cfg == GEMM_128x1 ? b.walkers : blocks);
    for (int i = 0; i < b.n; ++i) b.p[i].e.partial = partial;
    for (int i = 0; i < b.n_bias; ++i) { b.bias[i].partial = partial + n_partial; n_partial += b.bias[i].rows; }
  }
  const int mode0 = b.p[0].e.mode;
  const int kind = mode0 == EPI_WGRAD_NEUMANN ? BETTY_K_GEMM_UPDATE
                 : mode0 == EPI_WGRAD_NEUMANN_L2 ? BETTY_K_GEMM_UPDATE_FINAL
                 : (mode0 == EPI_RFWD || mode0 == EPI_RFWD_LAST || mode0 == EPI_RFWD_LAST_HESS) ? BETTY_K_GEMM_RFWD
                 : mode0 == EPI_RBWD ? BETTY_K_GEMM_RBWD : BETTY_K_GEMM;
  Launch l(ctx, kind, flops, bytes);
  hipError_t err = hipSuccess;
  if (elem == ELEM_BF16) launch_elem<__bf16>(cfg, b.p[0].e.mode, total, ctx.stream, b, err);
  else launch_elem<float>(cfg, b.p[0].e.mode, total, ctx.stream, b, err);
  if (err != hipSuccess && ctx.first_error == hipSuccess) ctx.first_error = err;
  return n_partial;
}

}  // namespace betty
