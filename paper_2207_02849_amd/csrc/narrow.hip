// Models whose layers are narrow: every layer of 16 samples in one workgroup.
//
// The forward, backward and forward-over-reverse chains couple layers, not samples; only the weight gradients sum
// over the batch.  As products of the whole batch they are one dependent launch per layer and direction, 4 to 5 us
// each whatever the width.  Here a workgroup takes 16 samples through the whole chain: the activations of the
// previous layer are an operand in LDS, weights come straight from memory into MFMA fragments, a layer costs two
// barriers.  Every workgroup reads all weights (the direction's too), which is what limits the width.
//
// A link (one layer, one direction) is 16 x n_out outputs: 16-tiles over the 8 wavefronts, K split over the
// wavefronts left over (partial tiles summed in order through LDS, as in gemm16_kernel).  Products with operands
// of the direction alone (a V, delta V^T), which do not wait for the layer before, come before the barrier.
#include "internal.h"

namespace betty {

constexpr int NW = 8, NT = 64 * NW, NROWS = NARROW_ROWS;

template <typename T> constexpr int narrow_ks() { return 64 / (int)sizeof(T); }     // elements of K per step
template <typename T> __device__ __forceinline__ T narrow_cast(float x) { return (T)x; }

// U steps of an operand row at this lane's chunk (beyond n they repeat the last one and are not multiplied)
template <typename T, int U>
__device__ __forceinline__ void narrow_load(const T* P, int s, int n, u32x4 (&f)[U]) {
  constexpr int KS = narrow_ks<T>();
#pragma unroll
  for (int u = 0; u < U; ++u) f[u] = *(const u32x4*)(P + (long long)(s + min(u, n - 1)) * KS);
}

// acc += A B^T over the steps [s0, s1); A, B in memory at this lane's row and chunk
template <typename T, int U>
__device__ __forceinline__ void narrow_mac(const T* A, const T* B, int s0, int s1, MfmaSum16<T>& acc) {
  for (int s = s0; s < s1; s += U) {
    const int n = min(U, s1 - s);
    u32x4 a[U], b[U];
    narrow_load<T, U>(A, s, n, a);
    narrow_load<T, U>(B, s, n, b);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) acc.step(a[u], b[u]);
  }
}
// ... with A in LDS and the first U steps of B already in w
template <typename T, int U>
__device__ __forceinline__ void narrow_mac_lds(const T* A, const T* B, int s0, int s1, u32x4 (&w)[U], MfmaSum16<T>& acc) {
  constexpr int KS = narrow_ks<T>();
  const int n0 = min(U, s1 - s0);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < n0) acc.step(*(const u32x4*)(A + (s0 + u) * KS), w[u]);
  for (int s = s0 + U; s < s1; s += U) {
    const int n = min(U, s1 - s);
    u32x4 b[U];
    narrow_load<T, U>(B, s, n, b);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) acc.step(*(const u32x4*)(A + (s + u) * KS), b[u]);
  }
}

// The operands of a link: products over the same K with A in memory (first two) and in LDS
template <typename T>
struct NarrowLink {
  const T* A1; const T* B1; const T* A2; const T* B2;    // A null: absent
  int lds; const T* B0;                                  // LDS buffer 0 or 1, or -1: absent
  NarrowSplit split;
  int lda, ldb, K, N;                                    // lda: of operands in memory
};

// pre(col, row) before the products, fin(col, row, acc) with four consecutive rows of one column; columns up to N
// rounded up to a step of K are finished (the next link reads them as padding).  Every thread calls it.  What pre reads
// it reads without conditions, at clamped positions: a register that is loaded on one path and set on another is waited
// for where the paths meet, and with it every store of the link before.
template <typename T, int U, typename Pre, typename Fin>
__device__ __forceinline__ void narrow_link_of(const NarrowLink<T>& k, const T* bufs, int pitch, int i0, float* red, Pre pre, Fin fin) {
  constexpr int KS = narrow_ks<T>(), EPC = 16 / (int)sizeof(T);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fc = (lane >> 4) * EPC;
  const int nt = (k.N + KS - 1) / KS * (KS / 16), S = (k.K + KS - 1) / KS, ks = k.split.ks;
  for (int base = 0; base < nt; base += NW) {
    const int kp = ks > 1 ? wave * k.split.by_nt >> 8 : 0, tile = ks > 1 ? wave - kp * nt : base + wave;
    const bool active = kp < ks && tile < nt;
    const int s0 = kp * k.split.per, s1 = min(S, s0 + k.split.per), col = tile * 16 + fr, row = 4 * (lane >> 4);
    MfmaSum16<T> sums;
    u32x4 w[U];
    if (active) {
      const long long b = (long long)(tile * 16 + fr) * k.ldb + fc;
      if (k.lds >= 0) narrow_load<T, U>(k.B0 + b, s0, min(U, s1 - s0), w);
      pre(min(col, k.N - 1), row);
      if (k.A1) narrow_mac<T, U>(k.A1 + (long long)(i0 + fr) * k.lda + fc, k.B1 + b, s0, s1, sums);
      if (k.A2) narrow_mac<T, U>(k.A2 + (long long)(i0 + fr) * k.lda + fc, k.B2 + b, s0, s1, sums);
    }
    if (base == 0) lds_barrier();
    if (active && k.lds >= 0)
      narrow_mac_lds<T, U>(bufs + k.lds * NROWS * pitch + fr * pitch + fc, k.B0 + (long long)(tile * 16 + fr) * k.ldb + fc, s0, s1, w, sums);
    f32x4v acc = sums.total();
    if (ks > 1) {
      if (active && kp > 0) *(f32x4v*)(red + ((kp - 1) * nt + tile) * 256 + lane * 4) = acc;
      lds_barrier();
      if (active && kp == 0)
        for (int q = 1; q < ks; ++q) acc += *(const f32x4v*)(red + ((q - 1) * nt + tile) * 256 + lane * 4);
    }
    if (active && kp == 0) {
      const float v[4] = {acc[0], acc[1], acc[2], acc[3]};
      fin(col, row, v);
    }
  }
}

template <typename T, typename Pre, typename Fin>
__device__ __forceinline__ void narrow_link(const NarrowLink<T>& k, const T* bufs, int pitch, int i0, float* red, Pre pre, Fin fin) {
  if (k.split.per == 1) narrow_link_of<T, 1>(k, bufs, pitch, i0, red, pre, fin);
  else if (k.split.per == 2) narrow_link_of<T, 2>(k, bufs, pitch, i0, red, pre, fin);
  else narrow_link_of<T, 4>(k, bufs, pitch, i0, red, pre, fin);
}

// transposed copy [column][sample] of an operand in LDS
template <typename T>
__device__ __forceinline__ void narrow_store_t(const T* buf, int pitch, T* out, int ldT, int i0, int N) {
  for (int x = threadIdx.x; x < N * 4; x += NT) {
    const int c = x >> 2, r = 4 * (x & 3);
    const float q[4] = {(float)buf[r * pitch + c], (float)buf[(r + 1) * pitch + c], (float)buf[(r + 2) * pitch + c], (float)buf[(r + 3) * pitch + c]};
    store4<T>(out + (long long)c * ldT + i0 + r, q);
  }
}

__device__ __forceinline__ float narrow_wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float narrow_wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

// the by-value argument block where it stands (captured or indexed as a parameter it would be copied to scratch)
template <typename A> __device__ __forceinline__ const A* narrow_args() { return (const A*)__builtin_amdgcn_kernarg_segment_ptr(); }

// TF: operand type of the forward products (fp32 beside bf16 for ReLU networks)
template <typename T, typename TF>
__global__ __launch_bounds__(NT) void narrow_grad_kernel(NarrowGradArgs) {
  const NarrowGradArgs& a = *narrow_args<NarrowGradArgs>();
  extern __shared__ u32x4 narrow_smem[];
  const NarrowNet& net = a.net;
  const int which = (int)blockIdx.x >= a.blocks0 ? 1 : 0, L = net.L, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const NarrowGradSide& sd = a.side[which];
  const int i0 = ((int)blockIdx.x - (which ? a.blocks0 : 0)) * NROWS, B = sd.B, pitch = net.pitch;
  auto fbuf = [&](int i) { return (TF*)narrow_smem + i * NROWS * pitch; };
  auto dbuf = [&](int i) { return (T*)narrow_smem + i * NROWS * pitch; };
  float* const zl = (float*)fbuf(2);
  float* const red = zl + NROWS * net.ldz;
  const int C = net.n[L];

  for (int l = net.first; l <= L; ++l) {
    const bool from_mem = l == net.first, last = l == L;
    const int N = net.n[l];
    NarrowLink<TF> k{};
    k.split = net.fwd[l - 1];
    k.lds = from_mem ? -1 : l & 1;
    k.A1 = from_mem ? (const TF*)(l == 1 ? sd.X : sd.A1) : nullptr;
    k.B0 = k.B1 = (const TF*)sd.Wf[l - 1];
    k.lda = k.ldb = net.np[l - 1]; k.K = net.n[l - 1]; k.N = N;
    const float* bl = sd.bias[l - 1];
    TF* const dst = fbuf((l + 1) & 1);
    T* const Ao = (T*)sd.A[l - 1];
    T* const At = (T*)sd.At[l - 1];
    float* const dp = sd.dphi[l - 1];
    float* const e2 = sd.e2[l - 1];
    const long long ldf = net.np[l];
    const float* bp = bl ? bl : (const float*)sd.P;              // (some address, where there is no bias)
    float bias;
    narrow_link<TF>(k, fbuf(0), pitch, i0, red,
      [&](int col, int) { bias = bp[col]; },
      [&](int col, int row, const float (&acc)[4]) {
        if (!bl) bias = 0.f;
        float d1[4], d2[4];
        if (last) {
#pragma unroll
          for (int r = 0; r < 4; ++r) if (col < C) zl[(row + r) * net.ldz + col] = acc[r] + bias;
          return;
        }
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          act_eval(net.act, acc[r] + bias, v[r], d1[r], d2[r]);
          if (col >= N) v[r] = 0.f;
          dst[(row + r) * pitch + col] = narrow_cast<TF>(v[r]);
          if (col >= N || i0 + row + r >= B) { v[r] = 0.f; continue; }
          const long long o = (i0 + row + r) * ldf + col;
          Ao[o] = narrow_cast<T>(v[r]);
          dp[o] = d1[r];
          if (e2) e2[o] = d2[r];
        }
        if (col < N) store4<T>(At + (long long)col * sd.Bp + i0 + row, v);
      });
  }
  lds_barrier();

  // loss, sample weight and output delta: a wavefront per sample, two samples each
  for (int row = wave; row < NROWS; row += NW) {
    const int i = i0 + row, iv = min(i, B - 1);
    const bool ok = i < B, ce = net.loss == BETTY_LOSS_SOFTMAX_CE;
    const Labels lab = *sd.labels;
    float* const z = zl + row * net.ldz;
    T* const D = dbuf(0) + row * pitch;
    float ell, m = 0.f, sum = 1.f;
    int y = 0;
    const float* t = ce ? nullptr : lab.target + (long long)iv * C;
    if (ce) {
      m = -INFINITY;
      for (int c = lane; c < C; c += 64) m = fmaxf(m, z[c]);
      m = narrow_wave_max(m);
      sum = 0.f;
      for (int c = lane; c < C; c += 64) sum += expf(z[c] - m);
      sum = narrow_wave_sum(sum);
      y = min(max(lab.y[iv], 0), C - 1);           // clamped into [0, C), for the gather and the one-hot alike
      ell = logf(sum) + m - z[y];
    } else {
      float acc = 0.f;
      for (int c = lane; c < C; c += 64) { const float r = z[c] - t[c]; acc += r * r; }
      ell = narrow_wave_sum(acc);
    }
    float omega = 1.f;
    if (sd.reweight && sd.omega_fixed) {
      omega = sd.omega_fixed[iv];
    } else if (sd.reweight) {
      const int H = a.hidden;
      float part = 0.f;
      for (int j = lane; j < H; j += 64)
        part += a.theta[2 * H + j] * fmaxf(a.theta[j] * ell + a.theta[H + j], 0.f);
      part = narrow_wave_sum(part) + a.theta[3 * H];
      omega = 1.f / (1.f + expf(-part));
      // sigmoid'(x) = sigmoid(x) sigmoid(-x): no 1 - omega, which loses every digit once omega rounds to 1
      if (ok && lane == 0 && sd.dsig) sd.dsig[i] = omega / (1.f + expf(part));
    }
    const float s = omega * sd.inv_batch, inv = 1.f / sum;
    if (ok && lane == 0) { sd.ell[i] = ell; sd.s[i] = s; sd.omega[i] = omega; }
    constexpr int KS = narrow_ks<T>();
    for (int c = lane; c < (C + KS - 1) / KS * KS; c += 64) {
      float dv = 0.f;
      if (ok && c < C) {
        const long long o = (long long)i * net.np[L] + c;
        sd.ZL[o] = z[c];
        if (ce) {
          const float p = expf(z[c] - m) * inv;
          sd.P[o] = p;
          dv = s * (p - (c == y ? 1.f : 0.f));
        } else {
          dv = s * 2.f * (z[c] - t[c]);
        }
        ((T*)sd.D[L - 1])[o] = narrow_cast<T>(dv);
      }
      D[c] = narrow_cast<T>(dv);
    }
  }
  lds_barrier();
  narrow_store_t<T>(dbuf(0), pitch, (T*)sd.Dt[L - 1], sd.Bp, i0, C);

  int from = 0;
  for (int l = L; l >= 2; --l, from ^= 1) {
    const int N = net.n[l - 1];
    const long long ldf = net.np[l - 1];
    NarrowLink<T> k{};
    k.split = net.bwd[l - 1];
    k.lds = from;
    k.B0 = (const T*)sd.Wn[l - 1];
    k.ldb = net.np[l]; k.K = net.n[l]; k.N = N;
    T* const dst = dbuf(from ^ 1);
    const float* dp = sd.dphi[l - 2];
    float* const e2 = sd.e2[l - 2];
    T* const D = (T*)sd.D[l - 2];
    T* const Dt = (T*)sd.Dt[l - 2];
    const float* ep = e2 ? e2 : dp;
    float d1[4], d2[4];
    narrow_link<T>(k, dbuf(0), pitch, i0, red,
      [&](int col, int row) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const long long o = min(i0 + row + r, B - 1) * ldf + col;
          d1[r] = dp[o];
          d2[r] = ep[o];
        }
      },
      [&](int col, int row, const float (&acc)[4]) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool ok = col < N && i0 + row + r < B;
          const long long o = (i0 + row + r) * ldf + col;
          v[r] = ok ? acc[r] * d1[r] : 0.f;
          if (ok && e2) e2[o] = acc[r] * d2[r];
          if (ok && D) D[o] = narrow_cast<T>(v[r]);
          if (l > 2) dst[(row + r) * pitch + col] = narrow_cast<T>(v[r]);
        }
        if (col < N) store4<T>(Dt + (long long)col * sd.Bp + i0 + row, v);
      });
  }
}

template <typename T>
__global__ __launch_bounds__(NT) void narrow_rop_kernel(NarrowRopArgs) {
  const NarrowRopArgs& a = *narrow_args<NarrowRopArgs>();
  extern __shared__ u32x4 narrow_smem[];
  const NarrowNet& net = a.net;
  const int L = net.L, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i0 = (int)blockIdx.x * NROWS, B = a.B, pitch = net.pitch, C = net.n[L];
  auto buf = [&](int i) { return (T*)narrow_smem + i * NROWS * pitch; };
  float* const zl = (float*)buf(2);
  float* const red = zl + NROWS * net.ldz;

  for (int l = net.first; l <= L; ++l) {
    const bool last = l == L;
    const int N = net.n[l];
    const long long ldf = net.np[l];
    NarrowLink<T> k{};
    k.split = net.fwd[l - 1];
    k.lds = l == net.first ? -1 : l & 1;
    k.A2 = l > 1 && l == net.first ? (const T*)a.RA1 : nullptr;
    k.B0 = k.B2 = (const T*)a.Wt[l - 1];
    k.A1 = (const T*)(l == 1 ? a.X : a.A[l - 2]);
    k.B1 = (const T*)a.Vt[l - 1];
    k.lda = k.ldb = net.np[l - 1]; k.K = net.n[l - 1]; k.N = N;
    T* const dst = buf((l + 1) & 1);
    const float* cbl = a.cbias[l - 1];
    const float* dphi = last ? a.P : a.dphi[l - 1];
    float* const Rz = a.Rz[l - 1];
    T* const RAt = (T*)a.RAt[l - 1];
    const float* cp = cbl ? cbl : a.P;                           // (some address, where there is none)
    float cb, dp[4];
    narrow_link<T>(k, buf(0), pitch, i0, red,
      [&](int col, int row) {
        cb = cp[col];
#pragma unroll
        for (int r = 0; r < 4; ++r) dp[r] = dphi[min(i0 + row + r, B - 1) * ldf + col];
      },
      [&](int col, int row, const float (&acc)[4]) {
        if (!cbl) cb = 0.f;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float z = acc[r] + cb;
          if (last) {
            if (col < C) zl[(row + r) * net.ldz + col] = z;
            continue;
          }
          const bool ok = col < N && i0 + row + r < B;
          v[r] = ok ? dp[r] * z : 0.f;
          dst[(row + r) * pitch + col] = narrow_cast<T>(v[r]);
          if (ok && Rz) Rz[(i0 + row + r) * ldf + col] = z;
        }
        if (!last && col < N && RAt) store4<T>(RAt + (long long)col * a.Bp + i0 + row, v);
      });
  }
  lds_barrier();

  // loss Hessian (or the loss's derivative along Rz): a wavefront per sample
  for (int row = wave; row < NROWS; row += NW) {
    const int i = i0 + row, iv = min(i, B - 1);
    const bool ok = i < B, ce = net.loss == BETTY_LOSS_SOFTMAX_CE;
    const float* z = zl + row * net.ldz;
    const float* p = a.P + (long long)iv * net.np[L];
    if (a.cvec) {
      const Labels lab = *a.labels;
      float acc = 0.f;
      if (ce) {
        for (int c = lane; c < C; c += 64) acc += p[c] * z[c];
        acc = narrow_wave_sum(acc);
        acc -= z[min(max(lab.y[iv], 0), C - 1)];
      } else {
        const float* zz = a.Z + (long long)iv * net.np[L];
        const float* t = lab.target + (long long)iv * C;
        for (int c = lane; c < C; c += 64) acc += 2.f * (zz[c] - t[c]) * z[c];
        acc = narrow_wave_sum(acc);
      }
      if (ok && lane == 0) a.cvec[i] = acc;
      continue;
    }
    const float si = a.s[iv];
    float dot = 0.f;
    if (ce) {
      for (int c = lane; c < C; c += 64) dot += p[c] * z[c];
      dot = narrow_wave_sum(dot);
    }
    constexpr int KS = narrow_ks<T>();
    for (int c = lane; c < (C + KS - 1) / KS * KS; c += 64) {
      float v = 0.f;
      if (ok && c < C) v = ce ? si * (p[c] * z[c] - p[c] * dot) : si * 2.f * z[c];
      buf(0)[row * pitch + c] = narrow_cast<T>(v);
    }
  }
  if (a.cvec) return;
  lds_barrier();
  narrow_store_t<T>(buf(0), pitch, (T*)a.RDt[L - 1], a.Bp, i0, C);

  int from = 0;
  for (int l = L; l >= 2; --l, from ^= 1) {
    const int N = net.n[l - 1];
    const long long ldf = net.np[l - 1];
    NarrowLink<T> k{};
    k.split = net.bwd[l - 1];
    k.lds = from;
    k.B0 = (const T*)a.Wn[l - 1];
    k.A1 = (const T*)a.D[l - 1];
    k.B1 = (const T*)a.Vn[l - 1];
    k.lda = k.ldb = net.np[l]; k.K = net.n[l]; k.N = N;
    T* const dst = buf(from ^ 1);
    const float* dphi = a.dphi[l - 2];
    const float* e2 = a.e2[l - 2];
    const float* Rz = a.Rz[l - 2];
    T* const RDt = (T*)a.RDt[l - 2];
    const float* ep = e2 ? e2 : dphi;
    const float* zp = e2 ? Rz : dphi;
    float dp[4], e2v[4], rz[4];
    narrow_link<T>(k, buf(0), pitch, i0, red,
      [&](int col, int row) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const long long o = min(i0 + row + r, B - 1) * ldf + col;
          dp[r] = dphi[o];
          e2v[r] = ep[o];
          rz[r] = zp[o];
        }
      },
      [&](int col, int row, const float (&acc)[4]) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = col < N && i0 + row + r < B ? e2 ? acc[r] * dp[r] + e2v[r] * rz[r] : acc[r] * dp[r] : 0.f;
          if (l > 2) dst[(row + r) * pitch + col] = narrow_cast<T>(v[r]);
        }
        if (col < N) store4<T>(RDt + (long long)col * a.Bp + i0 + row, v);
      });
  }
}

// ------------------------------------------------------------------------------------------
// The forward-over-reverse pass with everything a link needs in LDS before the chain begins.  narrow_rop_kernel fetches
// weights, direction products and elementwise factors link by link, a memory latency or two (1.6 us) in every link.
// Of these only the weights' product with the link before is in the chain.  So 16 wavefronts first form all products with
// operands of the direction alone (units: the 16-tiles of all links) and leave them with phi' and phi'' in LDS as they stand in the accumulators;
// forward and backward weights go straight to LDS meanwhile.  A link is then LDS reads, MFMA and one barrier.  LDS bounds the width:
// the weights in both orientations and 3 or 4 floats an element of every hidden layer.
//
// Bound by the instructions that a wavefront issues one after the other, at 4 cycles and more each: 13-64-64-1, fp32, 200
// samples (13 workgroups) 8.2 us, of which 1 us arguments and requests, 3.4 us the products along the direction, 1.8 us
// three forward links, 0.4 us the loss Hessian, 1.3 us two backward links; the launches per layer take 13.5 us,
// narrow_rop_kernel as much.  What counted: no loads or stores under conditions, 32-bit offsets from scalar bases, padding that
// is zero in memory instead of masks, small loops (first version, 3600 instructions: 12.5 us).  Eight 32-wide layers, bf16, 100 samples:
// product and weight gradient 30.7 -> 16.9 us.  Requesting a wavefront's next 16-tile ahead: 14.0 -> 14.5 us a step.
// ------------------------------------------------------------------------------------------

constexpr int SW = 16, ST = 64 * SW;                      // wavefronts, threads
constexpr int STAGED_LDS = 159 * 1024;

// elements of a matrix as the base, which stays in scalar registers, and 32 bits of offset
template <typename V, typename T> __device__ __forceinline__ V at32(const void* base, unsigned i) {
  return *(const V*)((const char*)base + i * (unsigned)sizeof(T));
}

// sums of U steps of A W^T from memory, all requested at once
template <typename T, int U>
__device__ __forceinline__ void staged_mac(const void* A, const void* W, unsigned a0, unsigned w0, MfmaSum16<T>& sums) {
  constexpr int KS = narrow_ks<T>();
  u32x4 a[U], w[U];
#pragma unroll
  for (int v = 0; v < U; ++v) { a[v] = at32<u32x4, T>(A, a0 + v * KS); w[v] = at32<u32x4, T>(W, w0 + v * KS); }
#pragma unroll
  for (int v = 0; v < U; ++v) sums.step(a[v], w[v]);
}
// ... from LDS
template <typename T, int U>
__device__ __forceinline__ void staged_mac_lds(const T* x, const T* w, MfmaSum16<T>& sums) {
  constexpr int KS = narrow_ks<T>();
  u32x4 a[U], b[U];
#pragma unroll
  for (int v = 0; v < U; ++v) { a[v] = *(const u32x4*)(x + v * KS); b[v] = *(const u32x4*)(w + v * KS); }
#pragma unroll
  for (int v = 0; v < U; ++v) sums.step(a[v], b[v]);
}

// CURV: phi'' is not zero
template <typename T, bool CURV>
__global__ __launch_bounds__(ST) void staged_rop_kernel(StagedArgs) {
  const StagedArgs& a = *narrow_args<StagedArgs>();
  extern __shared__ u32x4 narrow_smem[];
  char* const lds = (char*)narrow_smem;
  constexpr int KS = narrow_ks<T>(), EPC = 16 / (int)sizeof(T);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i0 = (int)blockIdx.x * NROWS, B = a.B, pitch = a.pitch, C = a.C;
  const int fr = lane & 15, fc = (lane >> 4) * EPC, row = 4 * (lane >> 4);
  T* const buf0 = (T*)(lds + a.buf);
  float* const zl = (float*)(lds + a.zl);
  const int ldz = a.ldz, Bp = a.Bp, n_fwd = a.n_fwd, n_bwd = a.n_bwd;
  auto buf = [&](int i) { return buf0 + i * NROWS * pitch; };
  auto slot = [&](int off, int tile) { return (f32x4v*)(lds + off + tile * 1024) + lane; };
  warm_lines<(sizeof(StagedArgs) + 63) / 64>();

  // All weights of the chain, straight to LDS.  A layer's rows are those of its outputs, a row K rounded up to a step (the
  // operands are zero there) and a chunk of room, which spreads the rows over the banks.
  {
    int q = 0;
    for (int g = wave; g < a.groups; g += SW) {
      while (q + 1 < a.n_w && g >= a.w[q + 1].group0) ++q;
      const StagedWeights& w = a.w[q];
      const int y = (g - w.group0) * 64 + lane, r = __umulhi(y, w.inv), c = y - r * w.cpr;
      const unsigned o = min(r, w.rows - 1) * w.ld + min(c, w.cpr - 2) * EPC;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)w.src + o * (unsigned)sizeof(T)),
                                       (__attribute__((address_space(3))) void*)(lds + g * 1024), 16, 0, 0);
    }
  }
  const int is = i0 + wave;                                // the sample whose loss Hessian this wavefront applies
  const float* const prow = a.P + (long long)is * a.ldp;
  const float p0 = prow[lane], s0 = a.s[is];

  // Products with operands of the direction alone.  phi' and phi'' are zero beyond the batch and beyond the layer's width, and so
  // is everything that leaves a link there.
  for (int u = wave; u < a.units; u += SW) {
    const int id = a.unit[u], tile = id >> 4, col = tile * 16 + fr;
    const StagedPart& p = a.part[id & 15];
    const unsigned a0 = (i0 + fr) * p.ld + fc, w0 = col * p.ld + fc, f0 = (i0 + row) * p.ldf + col;
    const float* const bp = p.bias ? p.bias : p.dphi;
    const float bias = bp[p.bias ? min(col, p.N - 1) : 0];
    f32x4v d = {}, e = {}, rz = {};
    if (p.D >= 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        d[k] = at32<float, float>(p.dphi, f0 + k * p.ldf);
        if (CURV) e[k] = at32<float, float>(p.e2, f0 + k * p.ldf);
      }
      if (CURV && p.finish) {
#pragma unroll
        for (int k = 0; k < 4; ++k) rz[k] = at32<float, float>(p.Rz, f0 + k * p.ldf);
      }
    }
    MfmaSum16<T> sums;
    for (int m = 0; m < p.products; ++m) {
      const void* const A = p.A[m];
      const void* const W = p.W[m];
      int s = 0;
      for (; s + 8 <= p.steps; s += 8) staged_mac<T, 8>(A, W, a0 + s * KS, w0 + s * KS, sums);
      if (p.steps & 4) { staged_mac<T, 4>(A, W, a0 + s * KS, w0 + s * KS, sums); s += 4; }
      if (p.steps & 2) { staged_mac<T, 2>(A, W, a0 + s * KS, w0 + s * KS, sums); s += 2; }
      if (p.steps & 1) staged_mac<T, 1>(A, W, a0 + s * KS, w0 + s * KS, sums);
    }
    f32x4v acc = sums.total();
    if (p.finish) acc = CURV ? acc * d + e * rz : acc * d;
    else if (p.bias) acc += bias;
    *slot(p.S, tile) = acc;
    if (p.D >= 0) *slot(p.D, tile) = d;
    if (CURV && p.E >= 0) *slot(p.E, tile) = e;
  }
  __syncthreads();

  // sums += the operand in LDS times the weights of a link
  auto mac = [&](const T* A, const StagedLink& k, int tile, MfmaSum16<T>& sums) {
    const T* x = A + fr * pitch + fc;
    const T* w = (const T*)(lds + k.w) + min(tile * 16 + fr, k.N - 1) * k.wpitch + fc;
    for (int s = k.steps >> 2; s > 0; --s, x += 4 * KS, w += 4 * KS) staged_mac_lds<T, 4>(x, w, sums);
    if (k.steps & 2) { staged_mac_lds<T, 2>(x, w, sums); x += 2 * KS; w += 2 * KS; }
    if (k.steps & 1) staged_mac_lds<T, 1>(x, w, sums);
  };

  auto tiles = [&](int n) { return (n + KS - 1) / KS * (KS / 16); };
  // a hidden layer's R z: R a as the next operand and for the weight gradients, phi'' R z beside what the backward link adds
  auto hidden = [&](const StagedLink& k, int tile, int to, const f32x4v& z) {
    const f32x4v d = *slot(k.D, tile);
    if (n_bwd > 0) {
      if (CURV) *slot(k.T, tile) = *slot(k.T, tile) * d + *slot(k.E, tile) * z;
      else *slot(k.T, tile) *= d;
    }
    const int col = tile * 16 + fr;
    T* const o = buf(to) + row * pitch + col;
    const float v[4] = {d[0] * z[0], d[1] * z[1], d[2] * z[2], d[3] * z[3]};
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r * pitch] = narrow_cast<T>(v[r]);
    if (col < k.N && k.outT) store4<T>((T*)k.outT + (col * Bp + i0 + row), v);
  };
  StagedLink k = a.fwd[0];
  for (int tile = wave; tile < tiles(k.N); tile += SW) hidden(k, tile, 1, *slot(k.F, tile));
  for (int i = 1; i < n_fwd - 1; ++i) {
    k = a.fwd[i];
    lds_barrier();
    for (int tile = wave; tile < tiles(k.N); tile += SW) {
      const f32x4v f = *slot(k.F, tile);
      MfmaSum16<T> sums;
      mac(buf(i & 1), k, tile, sums);
      hidden(k, tile, (i + 1) & 1, f + sums.total());
    }
  }
  k = a.fwd[n_fwd - 1];
  lds_barrier();
  for (int tile = wave; tile < tiles(k.N); tile += SW) {
    const f32x4v f = *slot(k.F, tile);
    MfmaSum16<T> sums;
    mac(buf((n_fwd - 1) & 1), k, tile, sums);
    const f32x4v z = f + sums.total();
    const int col = tile * 16 + fr;
    if (col < C) {
#pragma unroll
      for (int r = 0; r < 4; ++r) zl[(row + r) * ldz + col] = z[r];
    }
  }
  lds_barrier();

  // loss Hessian (or the loss's derivative along Rz): a wavefront per sample
  {
    const bool ok = is < B, ce = a.loss == BETTY_LOSS_SOFTMAX_CE;
    const float* z = zl + wave * ldz;
    auto p = [&](int c) { return c < 64 ? p0 : prow[c]; };
    if (a.cvec) {
      const int iv = min(is, B - 1);
      const Labels lab = *a.labels;
      float acc = 0.f;
      if (ce) {
        for (int c = lane; c < C; c += 64) acc += p(c) * z[c];
        acc = narrow_wave_sum(acc);
        acc -= z[min(max(lab.y[iv], 0), C - 1)];
      } else {
        const float* zz = a.Z + (long long)iv * a.ldp;
        const float* tg = lab.target + (long long)iv * C;
        for (int c = lane; c < C; c += 64) acc += 2.f * (zz[c] - tg[c]) * z[c];
        acc = narrow_wave_sum(acc);
      }
      if (ok && lane == 0) a.cvec[is] = acc;
      return;
    }
    float dot = 0.f;
    if (ce) {
      for (int c = lane; c < C; c += 64) dot += p(c) * z[c];
      dot = narrow_wave_sum(dot);
    }
    for (int c = lane; c < (C + KS - 1) / KS * KS; c += 64) {
      float v = 0.f;
      if (ok && c < C) v = ce ? s0 * (p(c) * z[c] - p(c) * dot) : s0 * 2.f * z[c];
      buf(0)[wave * pitch + c] = narrow_cast<T>(v);
    }
  }
  lds_barrier();
  for (int x = t; x < C * 4; x += ST) {                              // transposed copy
    const int c = x >> 2, r = 4 * (x & 3);
    const T* b = buf(0) + r * pitch + c;
    const float q[4] = {(float)b[0], (float)b[pitch], (float)b[2 * pitch], (float)b[3 * pitch]};
    store4<T>((T*)a.RDt + (long long)c * a.Bp + i0 + r, q);
  }

  for (int i = 0; i < n_bwd; ++i) {
    k = a.bwd[i];
    const bool last = i + 1 == n_bwd;
    for (int tile = wave; tile < tiles(k.N); tile += SW) {
      const f32x4v d = *slot(k.D, tile), tt = *slot(k.T, tile);
      MfmaSum16<T> sums;
      mac(buf(i & 1), k, tile, sums);
      const f32x4v x = sums.total() * d + tt;
      const int col = tile * 16 + fr;
      const float v[4] = {x[0], x[1], x[2], x[3]};
      if (!last) {
        T* const o = buf((i + 1) & 1) + row * pitch + col;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r * pitch] = narrow_cast<T>(v[r]);
      }
      if (col < k.N) store4<T>((T*)k.outT + (col * Bp + i0 + row), v);
    }
    if (!last) lds_barrier();
  }
}

// ------------------------------------------------------------------------------------------

constexpr size_t NARROW_LDS = 150 * 1024;

size_t narrow_lds(NarrowNet& net, Elem elem, bool wide) {
  const size_t es = wide || elem == ELEM_F32 ? 4 : 2;
  int w = 16;
  for (int l = 1; l <= net.L; ++l) w = w > net.n[l] ? w : net.n[l];
  // (an odd number of 16-byte chunks a row: the fragment reads of 16 rows spread over the banks)
  net.pitch = (w + 31) / 32 * 32 + 16 / (int)(elem == ELEM_F32 ? 4 : 2);
  net.ldz = (net.n[net.L] + 3) / 4 * 4 + 1;
  return 2 * NROWS * (size_t)net.pitch * es + NROWS * (size_t)((net.ldz + 3) / 4 * 4) * 4 + (size_t)NW * 256 * 4;
}

// How each link spreads over the wavefronts
static void narrow_splits(NarrowNet& net, int ks_fwd, int ks_bwd) {
  auto one = [&](int K, int N, int KS) {
    const int nt = (N + KS - 1) / KS * (KS / 16), S = (K + KS - 1) / KS;
    NarrowSplit s{1, 1, 0};
    while (nt * s.ks * 2 <= NW && s.ks * 2 <= S) s.ks *= 2;
    s.per = (S + s.ks - 1) / s.ks;
    s.by_nt = (256 + nt - 1) / nt;                 // wave * by_nt >> 8 = wave / nt for wave < 16, nt <= 8
    return s;
  };
  for (int l = net.first; l <= net.L; ++l) net.fwd[l - 1] = one(net.n[l - 1], net.n[l], ks_fwd);
  for (int l = 2; l <= net.L; ++l) net.bwd[l - 1] = one(net.n[l], net.n[l - 1], ks_bwd);
}

template <typename K, typename A>
static void narrow_launch(Ctx& ctx, K kernel, PerDevice& allowed, int blocks, size_t lds, const A& a) {
  const hipError_t e = allow_lds(allowed, (const void*)kernel, NARROW_LDS);
  if (e != hipSuccess) { if (ctx.first_error == hipSuccess) ctx.first_error = e; return; }
  kernel<<<blocks, NT, lds, ctx.stream>>>(a);
}

void launch_narrow_grad(Ctx& ctx, Elem elem, bool wide, NarrowGradArgs& a, int n_sides, double flops) {
  a.blocks0 = (a.side[0].B + NROWS - 1) / NROWS;
  const int blocks = a.blocks0 + (n_sides > 1 ? (a.side[1].B + NROWS - 1) / NROWS : 0);
  const size_t lds = narrow_lds(a.net, elem, wide);
  Launch l(ctx, BETTY_K_GEMM, flops);
  narrow_splits(a.net, elem == ELEM_F32 || wide ? 16 : 32, elem == ELEM_F32 ? 16 : 32);
  static PerDevice allowed[3];
  if (elem == ELEM_F32) narrow_launch(ctx, narrow_grad_kernel<float, float>, allowed[0], blocks, lds, a);
  else if (wide) narrow_launch(ctx, narrow_grad_kernel<__bf16, float>, allowed[1], blocks, lds, a);
  else narrow_launch(ctx, narrow_grad_kernel<__bf16, __bf16>, allowed[2], blocks, lds, a);
}

void launch_narrow_rop(Ctx& ctx, Elem elem, NarrowRopArgs& a, double flops) {
  const int blocks = (a.B + NROWS - 1) / NROWS;
  const size_t lds = narrow_lds(a.net, elem, false);
  Launch l(ctx, BETTY_K_GEMM_RFWD, flops);
  narrow_splits(a.net, elem == ELEM_F32 ? 16 : 32, elem == ELEM_F32 ? 16 : 32);
  static PerDevice allowed[2];
  if (elem == ELEM_F32) narrow_launch(ctx, narrow_rop_kernel<float>, allowed[0], blocks, lds, a);
  else narrow_launch(ctx, narrow_rop_kernel<__bf16>, allowed[1], blocks, lds, a);
}

bool staged_plan(const NarrowRopArgs& r, Elem elem, bool curvature, StagedArgs& a) {
  a = StagedArgs{};
  const NarrowNet& net = r.net;
  const int KS = elem == ELEM_F32 ? 16 : 32, EPC = elem == ELEM_F32 ? 4 : 8, L = net.L, first = net.first;
  const bool backward = !r.cvec;
  auto steps = [&](int n) { return (n + KS - 1) / KS; };
  auto tiles = [&](int n) { return steps(n) * (KS / 16); };
  int width = 16, place[2][NARROW_MAX_L + 1] = {};
  long long at = 0;
  for (int back = 0; back < 2; ++back)
    for (int l = back ? 2 : first + 1; l <= L && (!back || backward); ++l) {
      const int K = back ? net.n[l] : net.n[l - 1];
      StagedWeights& w = a.w[a.n_w++];
      w.src = back ? r.Wn[l - 1] : r.Wt[l - 1];
      w.ld = net.np[back ? l : l - 1]; w.rows = back ? net.n[l - 1] : net.n[l];
      w.cpr = steps(K) * KS / EPC + 1;
      w.inv = (unsigned)((1ULL << 32) / w.cpr + 1);      // (exact below 2^16 chunks)
      w.group0 = a.groups;
      place[back][l] = 1024 * a.groups;
      a.groups += (w.rows * w.cpr + 63) / 64;
      at = 1024LL * a.groups;
      if (at > STAGED_LDS) return false;
    }
  auto take = [&](long long bytes) { const long long o = at; at += (bytes + 15) / 16 * 16; return at > STAGED_LDS ? -1 : (int)o; };
  int F[NARROW_MAX_L + 1], D[NARROW_MAX_L + 1], T[NARROW_MAX_L + 1], E[NARROW_MAX_L + 1];
  for (int l = 1; l <= L; ++l) {
    const long long n = 1024LL * tiles(net.n[l]);
    const bool inner = l >= first, hidden = l < L;
    F[l] = inner ? take(n) : -1;
    D[l] = hidden && (inner || backward) ? take(n) : -1;
    T[l] = hidden && backward ? take(n) : -1;
    E[l] = hidden && backward && curvature && inner ? take(n) : -1;
    if (inner) width = width > net.n[l] ? width : net.n[l];
  }
  a.pitch = (width + 31) / 32 * 32 + EPC;                // (an odd number of chunks a row, as in narrow_lds)
  a.buf = take(2LL * NROWS * a.pitch * (16 / EPC));
  a.zl = take(4LL * NROWS * net.ldz);
  if (at > STAGED_LDS) return false;
  a.bytes = (int)at;
  int n = 0;
  auto part = [&](const void* A, const void* W, int K, int N, int ld, int out, int S, int D, int E, int fin) -> StagedPart& {
    StagedPart& p = a.part[n];
    for (int tile = 0; tile < tiles(N); ++tile, ++a.units)
      if (a.units < STAGED_UNITS) a.unit[a.units] = (unsigned short)(tile << 4 | n);
    ++n;
    const float* any = r.P;
    p = StagedPart{{A, A}, {W, W}, nullptr, any, any, any, ld, steps(K), N, net.np[out], 1, S, D, E, fin};
    if (out < L && r.dphi[out - 1]) p.dphi = p.e2 = p.Rz = r.dphi[out - 1];
    if (E >= 0 || fin == 2) p.e2 = r.e2[out - 1];
    if (fin == 2) p.Rz = r.Rz[out - 1];
    return p;
  };
  for (int l = first; l <= L; ++l) {
    StagedPart& p = part(l == 1 ? r.X : r.A[l - 2], r.Vt[l - 1], net.n[l - 1], net.n[l], net.np[l - 1], l, F[l], D[l], E[l], 0);
    p.bias = r.cbias[l - 1];
    if (l == 2 && first == 2) { p.A[1] = r.RA1; p.W[1] = r.Wt[1]; p.products = 2; }
    StagedLink& k = a.fwd[a.n_fwd++];
    k = StagedLink{l < L ? r.RAt[l - 1] : nullptr, place[0][l], 0, steps(net.n[l - 1]), net.n[l], F[l], D[l], T[l], E[l]};
    k.wpitch = (k.steps * KS / EPC + 1) * EPC;
  }
  for (int l = L; l >= 2 && backward; --l) {
    const bool whole = l - 1 < first;                    // R z of the layer that leaves is in memory already
    part(r.D[l - 1], r.Vn[l - 1], net.n[l], net.n[l - 1], net.np[l], l - 1, T[l - 1], whole ? D[l - 1] : -1, -1, whole ? curvature ? 2 : 1 : 0);
    StagedLink& k = a.bwd[a.n_bwd++];
    k = StagedLink{r.RDt[l - 2], place[1][l], 0, steps(net.n[l]), net.n[l - 1], -1, D[l - 1], T[l - 1], -1};
    k.wpitch = (k.steps * KS / EPC + 1) * EPC;
  }
  if (a.units > STAGED_UNITS) return false;
  a.B = r.B; a.Bp = r.Bp; a.C = net.n[L]; a.ldz = net.ldz; a.loss = net.loss; a.ldp = net.np[L];
  a.P = r.P; a.s = r.s; a.Z = r.Z; a.labels = r.labels; a.cvec = r.cvec; a.RDt = r.RDt[L - 1];
  return true;
}

void launch_staged_rop(Ctx& ctx, Elem elem, bool curvature, const StagedArgs& a, double flops) {
  const int blocks = (a.B + NROWS - 1) / NROWS;
  Launch l(ctx, BETTY_K_GEMM_RFWD, flops);
  static PerDevice allowed[4];
  auto go = [&](auto kernel, PerDevice& ok) {
    const hipError_t e = allow_lds(ok, (const void*)kernel, STAGED_LDS);
    if (e != hipSuccess) { if (ctx.first_error == hipSuccess) ctx.first_error = e; return; }
    kernel<<<blocks, ST, a.bytes, ctx.stream>>>(a);
  };
  if (elem == ELEM_F32) curvature ? go(staged_rop_kernel<float, true>, allowed[0]) : go(staged_rop_kernel<float, false>, allowed[1]);
  else curvature ? go(staged_rop_kernel<__bf16, true>, allowed[2]) : go(staged_rop_kernel<__bf16, false>, allowed[3]);
}

}  // namespace betty
