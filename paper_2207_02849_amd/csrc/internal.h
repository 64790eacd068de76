// Internal declarations shared by the translation units of libbetty_hip.so.
// Nothing here is part of the public ABI (see include/betty_hip.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "betty_hip.h"
#include "per_device.h"

namespace betty {

// Every operand matrix of a GEMM lives in the workspace as [rows_p][k_p] with both extents
// rounded up to PAD and the padding zero-filled, so the GEMM main loop needs no bounds
// checks.  PAD is a multiple of every tile extent used by the kernels.
constexpr int PAD = 128;
inline int padup(int n) { return (n + PAD - 1) / PAD * PAD; }

enum Elem { ELEM_F32 = 0, ELEM_BF16 = 1 };
inline size_t elem_size(Elem e) { return e == ELEM_F32 ? 4 : 2; }

// Accumulators = sum over up to two operand pairs of A_p (M x K_p) * B_p^T (B_p is N x K_p).
// Both operands are "K-major": element (row, k) at base[row * ld + k].
struct GemmArgs {
  const void* A[2];
  const void* B[2];
  int lda[2], ldb[2];        // leading dimensions in elements
  int K[2];                  // reduction extents in elements (operands are zero beyond them); 0 = pair absent
  // A holds bf16 value and remainder (EPI_GRAM): every 64 elements of K are followed by the 64 remainders,
  // both multiplied with the same 64 elements of B.  (EPI_WGRAD_SCALED: A of the first pair and B of the second do.)
  int split;
  int M, N;                  // valid output extent: defines the tile grid; epilogue stores are bounds-checked against it
  // Workgroups go to the eight XCDs round-robin, so tiles t, t+8, t+16, ... of a problem share an
  // L2.  With xgm x xgn = 8 those tiles are laid out as one compact (tiles_m/xgm) x (tiles_n/xgn)
  // rectangle, which cuts the operand panels each L2 has to fetch; 0 = row-major tile order.
  int xgm, xgn;
};

// What happens to a finished accumulator tile.
enum EpiMode {
  // Layer 1 at both points of a central difference (finite differences, fp32): t = alpha (acc + colvec), acc = X V_1,
  // z+- = e +- Rz[0] t with e = z_1 at w and Rz[0] the step on the device; out, outT, dphi_out take the plus point's
  // phi(z), phi'(z), out2, outT2 (fp32 here), d2_out the minus point's
  EPI_FWD_PM = 0,
  EPI_FWD = 1,             // z = acc + bias; out = phi(z); dphi_out = phi'(z); d2_out = phi''(z); with fp32 operands f0 = z if given
  EPI_FWD_LAST,          // f0 = acc + bias                       (logits)
  EPI_BWD,               // out = acc * dphi; e_io = acc * e_io   (delta of the layer below)
  EPI_RFWD,              // f0 = rz = acc + cbias (+ e); out = dphi * rz
  EPI_RFWD_LAST,         // f0 = acc + cbias (+ e)
  EPI_RBWD,              // out = (acc (+ e_io)) * dphi + e * Rz;  problems of mode GRAM may share the launch
  // Last layer of the R-forward with the loss Hessian applied in place (outputs of at most 32
  // columns, so that one MFMA block holds whole rows): rz = acc + cbias;
  // out = e[row] * (dphi .* rz - dphi * <dphi, rz>_row) for softmax cross-entropy (dphi = the
  // softmax probabilities, e = the per-sample scale), out = 2 e[row] rz for the squared error;
  // `act` carries the loss kind.
  EPI_RFWD_LAST_HESS,
  // The series in sample space (see neumann_samples_seq):
  //  GRAM    out = acc + gamma: a matrix over pairs of samples as the A operand of a later product; with bf16
  //          operands as value + remainder (GemmArgs::split), which carries 16 bits of it
  //  SAMPLE  f0 = s = g + beta x - alpha acc + colvec  (g = Rz, x = e, each may be null);
  //          out, outT = dphi .* s when asked for
  EPI_GRAM, EPI_SAMPLE,
  EPI_WGRAD,             // C = acc (+ 2 exp(lam) (x - p))                 flat parameter layout; p (an anchor) may be null
  EPI_WGRAD_INIT,        // v = acc (and p = acc when p is given); out = operand copies
  // One step of the Neumann partial sum in nested form, s_{j+1} = g + (I - alpha H) s_j with s_0 = g
  // (the same sum_{i<=j} (I - alpha H)^i g as the term-by-term recurrence, one state vector instead
  // of two): s is read from x, g from v;  Hs = acc (+ 2 exp(lam) s);  p = g + s - alpha Hs;  out =
  // operand copies of the new s.
  EPI_WGRAD_NEUMANN,
  EPI_WGRAD_NEUMANN_L2,  // last step for L2 decay: s read from p, new s kept in registers, C = -2 exp(lam) x (alpha s)
  EPI_WGRAD_SCALED,      // C = beta x - alpha acc
  // One step of the finite-difference series, acc = difference of the two perturbed gradients' data terms:
  // Hv = acc / (2 eps) (+ 2 exp(lam) v);  v <- v - alpha Hv;  p <- p + v.  _LAST: only the mixed VJP leaves,
  // C = -2 exp(lam) x (alpha p) (fd_mixed_l2), or 2 exp(lam) (alpha p) without x
  EPI_WGRAD_FD, EPI_WGRAD_FD_LAST,
  EPI_WGRAD_CG,          // C = acc (+ 2 exp(lam) x); the launch's sum is <x, C>
  EPI_WGRAD_SGD          // g = acc (+ 2 exp(lam) p) + gamma p; v <- beta v + g; p <- p - alpha v  (p = w, v = momentum)
};

struct Epilogue {
  int mode, act;
  const float* colvec;                   // per-column addend (bias or bias direction), may be null
  void* out; int ld;                     // operand-typed, row-major [row][col]
  int ldT; void* outT;                   // operand-typed, transposed [col][row]
  union {
    struct {                             // activation-shaped modes
      float* f0;                         // fp32 [row * ldf + col]
      float* dphi_out; float* d2_out;
      const float* dphi; float* e_io; const float* e; const float* Rz;
      long long ldf;
      void* out2; void* outT2;           // EPI_FWD: further copies of `out` in bf16 (same ld, ldT), or null; EPI_FWD_PM
    };
    struct {                             // parameter-shaped modes
      float* C; long long ldc;           // fp32 row-major (flat parameter slice)
      const float* lam; const float* x;  // same indexing as C
      float* v; float* p;
      const float* eps;                  // EPI_WGRAD_FD: device scalar
      // Sums that leave beside the result, one number per finishing wavefront (4 blockIdx.x + wavefront; bias
      // rows: BiasJob::partial): WGRAD exp(lam) (x - p)^2, INIT acc^2, FD the new v^2 (or p^2: sum_p).  May be null.
      // At most 64 terms are added in fp32 (a lane's share of a tile), everything beyond in double.
      double* partial;
      int sum_p;
    };
  };
  float alpha, beta, gamma;
};

struct GemmProblem { GemmArgs g; Epilogue e; };

// out[row] from sum_k Mt[row][k]: bias-shaped slices of the WGRAD modes
struct BiasJob {
  const void* Mt; int ld, rows, k, mode;
  const void* Mt2;                       // a second matrix whose sums are added, or null
  float* C; const float* lam; const float* x; float* v; float* p; float alpha, beta, gamma;
  const float* eps; double* partial; int sum_p;
};

constexpr int MAX_PROBLEMS = 8;
constexpr int GEMM_NCH = 8;              // 16-byte chunks per row of a k-tile
// tile extent x number of K groups per workgroup; a group is 2 x 2 wavefronts, except in 32x8 and 32x4
// (32-tile, groups of one wavefront) and 16 (16-tile, 4 to 16 groups of one wavefront)
enum { GEMM_128x1 = 0, GEMM_64x1 = 2, GEMM_64x2 = 3, GEMM_32x8 = 4, GEMM_128x64 = 5, GEMM_16 = 6, GEMM_32x4 = 7 };

// Assembled on the host and passed to the kernels by value, in a form cut to the kind of launch.
// Activation-shaped launches have few problems (train and validation batch; a link of the R-backward chain
// with matrices over samples, mode GRAM, beside it) and no bias rows; their short form costs the host less to launch (2.7 us against 4.5 us outside a graph).
template <int NP, int NB> struct GemmBatchT {
  int n = 0, n_bias = 0, gemm_blocks = 0;
  int walkers = 0;                       // wgrad128_kernel: workgroups that walk the tiles (set by launch_gemm_batch)
  int block_begin[NP + 1];
  int bias_begin[NB + 1];
  GemmProblem p[NP];
  BiasJob bias[NB > 0 ? NB : 1];
};
constexpr int MAX_SAMPLE_PROBLEMS = 16, MAX_CHAIN_PROBLEMS = 4;
typedef GemmBatchT<MAX_SAMPLE_PROBLEMS, MAX_PROBLEMS> GemmBatch;
typedef GemmBatchT<MAX_PROBLEMS, MAX_PROBLEMS> WgradBatch;
typedef GemmBatchT<MAX_SAMPLE_PROBLEMS, 0> SampleBatch;
typedef GemmBatchT<MAX_CHAIN_PROBLEMS, 0> ChainBatch;
static_assert(sizeof(WgradBatch) <= 3840 && sizeof(SampleBatch) <= 3840, "passed by value as kernel arguments (4 KiB limit)");

// Launch context: stream + optional per-launch event timing.
struct ProfRec { int kind; double flops, bytes; hipEvent_t e0, e1; float ms; };
struct Ctx {
  hipStream_t stream = nullptr;
  bool profiling = false;
  std::vector<ProfRec> recs;
  hipError_t first_error = hipSuccess;
  unsigned long long launches = 0;
  void begin(int kind, double flops, double bytes);
  void end();
};

struct Launch {   // RAII bracket around one kernel launch
  Ctx& c;
  Launch(Ctx& ctx, int kind, double flops = 0, double bytes = 0) : c(ctx) { c.begin(kind, flops, bytes); }
  ~Launch() { c.end(); }
};

// Allows a kernel that much dynamic LDS on the current device (the limit is kept per kernel and device).
inline hipError_t allow_lds(PerDevice& allowed, const void* kernel, size_t bytes) {
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess)
    allowed.once(device, [&]() {
      e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
      return e == hipSuccess;
    });
  return e;
}

// One 16-byte chunk of K for a 32 x 32 MFMA block: 8 bf16 (one v_mfma_f32_32x32x16_bf16) or 4 floats
// (four v_mfma_f32_32x32x2_f32).  Lane l supplies row l % 32 of A and of B; lanes 0-31 hold the
// even chunks of a chunk pair, lanes 32-63 the odd ones.  Register r of lane l of the result holds
// C[8*(r/4) + 4*(l/32) + r%4][l%32].
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // one 16-byte chunk

template <typename T> struct MfmaChunk;

template <> struct MfmaChunk<__bf16> {
  static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                  acc, 0, 0, 0);
  }
};

template <> struct MfmaChunk<float> {
  static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
};

// The same for a 16 x 16 block and 64 bytes of K: lane l supplies row l % 16 and chunk l / 16 of A and of B; register r of
// lane l of the result holds C[4*(l/16) + r][l%16].
typedef float f32x4v __attribute__((ext_vector_type(4)));
template <typename T> struct MfmaStep16;
template <> struct MfmaStep16<__bf16> {
  static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x4v& acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  }
};
template <> struct MfmaStep16<float> {
  static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x4v& acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
};

// Accumulators of a 16-tile.  In fp32 the four MFMA instructions of a step have one each, added at the end.  In the kernels of narrow
// models one chain of K additions, where those of whole batches add up partial sums of a few steps, left results 7 to 18 % further off
// fp64 than theirs (70 models: first-order passes, products, series, differences; up to 2.2 times with a long first
// layer), two 0 to 7 %; with four they are 2 to 8 % nearer, and a call takes 1 % longer.
template <typename T> struct MfmaSum16 {
  f32x4v a = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ void step(const u32x4& x, const u32x4& y) { MfmaStep16<T>::run(x, y, a); }
  __device__ __forceinline__ f32x4v total() const { return a; }
};
template <> struct MfmaSum16<float> {
  f32x4v a[4] = {};
  __device__ __forceinline__ void step(const u32x4& x, const u32x4& y) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[i]), __uint_as_float(y[i]), a[i], 0, 0, 0);
  }
  __device__ __forceinline__ f32x4v total() const { return (a[0] + a[1]) + (a[2] + a[3]); }
};

__device__ __forceinline__ void act_eval(int act, float z, float& a, float& d1, float& d2) {
  if (act == BETTY_ACT_RELU) {
    const bool pos = z > 0.f;
    a = pos ? z : 0.f; d1 = pos ? 1.f : 0.f; d2 = 0.f;
  } else if (act == BETTY_ACT_GELU_ERF) {
    const float Phi = 0.5f * (1.f + erff(z * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * expf(-0.5f * z * z);
    a = z * Phi; d1 = Phi + z * pdf; d2 = pdf * (2.f - z * z);
  } else {
    a = z; d1 = 1.f; d2 = 0.f;
  }
}

template <typename T> __device__ __forceinline__ void store1(T* p, float x);
template <> __device__ __forceinline__ void store1<float>(float* p, float x) { *p = x; }
template <> __device__ __forceinline__ void store1<__bf16>(__bf16* p, float x) { *p = (__bf16)x; }

// four consecutive elements, p aligned to 4 elements
template <typename T> __device__ __forceinline__ void store4(T* p, const float (&x)[4]);
template <> __device__ __forceinline__ void store4<float>(float* p, const float (&x)[4]) {
  *(float4*)p = make_float4(x[0], x[1], x[2], x[3]);
}
template <> __device__ __forceinline__ void store4<__bf16>(__bf16* p, const float (&x)[4]) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
  bf16x4 v = {(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
  *(bf16x4*)p = v;
}

// A barrier for what is exchanged through LDS: loads and stores of memory stay in flight across it (where nothing that goes to memory is
// read by another thread of the launch).  __syncthreads() waits for all of them, one to two microseconds.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Requests the first N 64-byte lines of the kernel arguments at once.  They are read all through a kernel, and the first scalar
// load from each would wait for memory where it stands, one after the other.
template <int N> __device__ __forceinline__ void warm_lines() {
  static_assert(N <= 60, "lines");
  const unsigned* p = (const unsigned*)__builtin_amdgcn_kernarg_segment_ptr();
  auto line = [&](int i) { return p[(i < N ? i : N - 1) * 16]; };
#define BETTY_W5(i_) "s"(line(i_)), "s"(line(i_ + 1)), "s"(line(i_ + 2)), "s"(line(i_ + 3)), "s"(line(i_ + 4))
  asm volatile("" :: BETTY_W5(0), BETTY_W5(5), BETTY_W5(10), BETTY_W5(15), BETTY_W5(20), BETTY_W5(25));
  if constexpr (N > 30) asm volatile("" :: BETTY_W5(30), BETTY_W5(35), BETTY_W5(40), BETTY_W5(45), BETTY_W5(50), BETTY_W5(55));
#undef BETTY_W5
}

// The mixed term of finite differences for L2 decay, -2 exp(lam) w q with q = alpha p: the central difference
// of grad_lambda along q, formed in double and rounded once.
__device__ __forceinline__ float fd_mixed_l2(float lam, float w, float alpha, float p) {
  return (float)(-2.0 * exp((double)lam) * (double)w * ((double)alpha * (double)p));
}

// ---- gemm.hip
int gemm_cfg_tile(int cfg);
// `partial` (weight-gradient launches): where their sums go, written into the batch; returns how many there are
int launch_gemm_batch(Ctx& ctx, Elem elem, int cfg, GemmBatch& batch, double algorithmic_flops,
                      double algorithmic_bytes = 0, double* partial = nullptr);

// ---- kernels.hip : operand conversion -----------------------------------------------------
// Where the labels or targets of a batch are: kept in the workspace and read by the kernels, so that a
// recorded launch sequence stays valid when another batch is registered.
struct Labels { const int32_t* y; const float* target; };

// out ([rows][ld], operand type), outT ([cols][ldT], operand type), out32, outT32 (the same in fp32) =
// convert(src[r * lds + c]); each may be null
struct ConvertJob {
  const float* src; long long lds; int rows, cols;
  void* out; int ld; void* outT; int ldT;
  float* out32 = nullptr; float* outT32 = nullptr;
};
// (Passed by value; a launch of up to four matrices takes a form of 0.3 KB, not 1.1: a minibatch registered and one SGD
// step of 1024-512-512-10 64.0 -> 63.7 us, the reweighting step of that model waited for 225.7 -> 223.2 us.)
constexpr int MAX_CONVERTS = 16, FEW_CONVERTS = 4;
template <int N> struct ConvertBatchT {
  int n = 0;
  int block_begin[N + 1];
  ConvertJob j[N];
  Labels* table = nullptr;     // the launch also writes labels[0], labels[1] to table[0], table[1] if given
  Labels labels[2];
};
typedef ConvertBatchT<MAX_CONVERTS> ConvertBatch;
void launch_convert_batch(Ctx&, Elem, ConvertBatch&);

// out+, out- = w + e v, w - e v as fp32 GEMM operands (as stored and transposed) with e = eps_scale /
// (|scale| sqrt(sum of partial)) times scale, and the bias slices as they are; e (without scale) also goes to *eps.
// w null: outT[0] = v, transposed, and nothing else
struct PerturbJob {
  const float* w; const float* v; int rows, cols;
  float* out[2]; int ld; float* outT[2]; int ldT;
  const float* b; const float* bv; float* bout[2];       // bias slices (cols entries), or null
};
struct PerturbBatch { int n = 0; int block_begin[MAX_PROBLEMS + 1]; PerturbJob j[MAX_PROBLEMS]; const float* eps; float scale; int signs;
  const double* partial; int n_partial; float eps_scale; float* eps_out; };   // eps null: every block forms it from the partial sums
void launch_perturb(Ctx&, PerturbBatch&);
// *eps = eps_scale / (|scale| sqrt(sum of n partial)), 0 if that sum is 0
void launch_fd_eps(Ctx&, const double* partial, int n, float eps_scale, float scale, float* eps);

// Weighted sum over the steps of the series: sum = beta sum + r (sum = r on the first step), n elements each, a
// multiple of 2048.  On the last step the result becomes an operand: in fp32 it goes back to r, in bf16 it takes the
// place of sum as value and remainder (GemmArgs::split).
struct AccumulateJob { void* r; float* sum; float beta; size_t n; };
struct AccumulateBatch { int n = 0; int block_begin[MAX_PROBLEMS + 1]; AccumulateJob j[MAX_PROBLEMS]; bool first, last; };
void launch_accumulate(Ctx&, Elem, AccumulateBatch&);

// ---- kernels.hip : loss rows ---------------------------------------------------------------
struct LossArgs {
  int loss, reweight, hidden;
  const float* Z; long long ldz;        // logits [rows][ldz]
  const Labels* labels; int C;
  const float* theta;                   // weight net (reweight only)
  const float* omega_fixed;             // reweight only: use these weights instead of R(l_i; theta)
  int rows; float inv_batch;             // (negative: the output delta with the opposite sign)
  float* ell; float* s; float* omega;   // per-sample outputs
  float* dsig;                          // omega_i (1 - omega_i), formed without cancellation (weight net evaluated here only)
  float* P;                             // softmax probabilities [rows][ldz] (CE)
  void* D; int ldD; void* Dt; int ldDt;  // s_i * dl_i/dz as GEMM operands, both orientations
};
struct LossBatch { int n = 0; LossArgs a[2]; };     // up to two batches (train, validation) per launch
void launch_loss_rows(Ctx&, Elem, const LossBatch&);
// Rdelta_L (fp32) = s_i * (d^2 l_i/dz^2) Rz_i
// The last layer of the R-op passes when the network output is narrow (at most 16 columns): one
// launch computes Rz_L = Ra_{L-1} W_L + a_{L-1} V_L + c_L, applies the loss Hessian (R delta_L) and
// propagates through the last layer, R delta_{L-1} = (R delta_L W_L^T + delta_L V_L^T) .* phi'
// + e2 .* Rz_{L-1}, with plain vector arithmetic (the products have 16 or fewer columns or
// reduction terms, a poor fit for 32-wide MFMA tiles).
struct LastRopArgs {
  const void* RA; const void* A; int lda;               // Ra_{L-1}, a_{L-1}: [B][n_in_p], operand type
  const void* Wt; const void* Vt; int ldt;              // W_L, V_L as [n_out_p][n_in_p]
  const void* Wn; const void* Vn; int ldn;              // W_L, V_L as [n_in_p][n_out_p]
  const float* cbias;                                   // bias direction of the last layer, or null
  // Direction products formed elsewhere (the series in sample space): AS = a_{L-1} V_L + c_L [B][ldas] and
  // DS = delta_L V_L^T [B][ldf] instead of A, Vt, Vn and cbias; null otherwise
  const float* AS; int ldas; const float* DS;
  const float* P; const float* s; int ldp;              // softmax probabilities [B][ldp], per-sample scale
  const void* DL; int ldd;                              // delta_L [B][ldd], operand type
  const float* dphi; const float* e2; const float* Rz; int ldf;   // layer L-1, fp32 [B][ldf]; e2 may be null
  void* RDL; void* RDLt; int ldRDLt;                    // out: R delta_L [B][ldd] and [n_out_p][ldRDLt]
  void* RD; int ldRD; void* RDt; int ldRDt;             // out: R delta_{L-1} [B][ldRD] (or null) and [n_in_p][ldRDt]
  int B, n_in, C, loss;
  // Directional form (cvec non-null): only c_i = <dl_i/dz, Rz_L,i> per sample leaves the kernel
  // (the per-sample directional derivative of the loss, for the reweighting mixed term);
  // labels / (Z, targets) give dl/dz for cross-entropy / squared error.
  float* cvec; const Labels* labels; const float* Z;
};
constexpr int LAST_ROP_MAX_C = 16;
void launch_last_layer_rop(Ctx&, Elem, const LastRopArgs&);

// The first-order counterpart for narrow outputs: logits z_L = a_{L-1} W_L + b_L, per-sample loss,
// sample weight and output delta (what loss_rows_kernel computes), and
// delta_{L-1} = (delta_L W_L^T) .* phi'(z_{L-1}) (with e2 <- (delta_L W_L^T) .* e2 in place when e2
// is given), for up to two batches (train, validation) in one launch.
struct LastGradSide {
  const void* A; int lda;                        // a_{L-1} [B][lda], operand type
  const Labels* labels;                          // labels, or targets [B][C]
  const float* omega_fixed;                      // sample weights to use instead of the weight net, or null
  float* ZL; float* P; int ldz;                  // out: logits, softmax probabilities, fp32 [B][ldz]
  float* ell; float* s; float* omega;            // out: per-sample loss, scale, weight
  float* dsig;                                   // out: omega (1 - omega) without cancellation (weight net evaluated here only)
  void* DL; void* DLt; int ldd, ldDLt;           // out: delta_L [B][ldd] and [n_out_p][ldDLt]
  const float* dphi; float* e2; int ldf;         // layer L-1, fp32 [B][ldf]
  void* D; int ldD; void* Dt; int ldDt;          // out: delta_{L-1} [B][ldD] (or null) and [n_in_p][ldDt]
  const void* Wt; const void* Wn;                // W_L as [n_out_p][n_in_p] and [n_in_p][n_out_p]
  const float* bias;                             // b_L (fp32), or null
  int B, reweight; float inv_batch;              // (inv_batch negative: the output delta with the opposite sign)
};
struct LastGradArgs {
  LastGradSide side[2]; int n_sides;
  int ldt, ldn;
  const float* theta; int hidden;                     // weight net (sides with reweight set)
  int n_in, C, loss;
};
void launch_last_layer_grad(Ctx&, Elem, const LastGradArgs&);

void launch_loss_hessian_rows(Ctx&, Elem, int loss, const float* P, const float* Rz, long long ld,
                              const float* s, int rows, int C, void* D, int ldD, void* Dt, int ldDt);
// c_i = < dl_i/dz, Rz_i >
void launch_loss_directional_rows(Ctx&, int loss, const float* P, const float* Z, const Labels* labels, const float* Rz, long long ld, int rows,
                                  int C, float* c);
// out = -(1/B) sum_i c_i dR(l_i; theta)/dtheta
// (c_minus given: c_i = (c_i - c_minus_i) / (2 eps), 0 if eps is 0: losses at two perturbed points)
void launch_wnet_theta_vjp(Ctx&, const float* ell, const float* dsig, const float* c, const float* c_minus, const float* eps,
                           const float* theta, int hidden, int rows, float inv_batch, float* out);

// ---- kernels.hip : flat parameter-shaped vectors ------------------------------------------
void launch_fill_zero(Ctx&, void* p, size_t bytes);
// (fd: formed in double, fd_mixed_l2)
void launch_mixed_l2(Ctx&, const float* lam, const float* w, const float* p, float alpha, float* out, size_t n, bool fd = false);
// out = 2 exp(logrho) (alpha p): the mixed VJP of the proximal cost into its anchor
void launch_mixed_prox(Ctx&, const float* logrho, const float* p, float alpha, float* out, size_t n);
void launch_fill_value(Ctx&, float* p, float value, size_t n);
// Conjugate gradient, two launches a step beside the Hessian product Hd (scalars stay on the device):
//  step  a = rs / <d, Hd> (0 if either is 0);  q += a d (q = a d in the first step);  r -= a Hd; leaves the partial
//        sums of <r, r>.  In the first step rs is the sum of rs_partial and goes to *rs.  With `out`, the last
//        step, only q and the mixed VJP leave: out = -2 exp(lam) w q, or 2 exp(lam) q without w
//  dir   d = r + (rs_new / rs) d (d = r if rs is 0) with rs_new = the partial sums, also to *rs_new; d leaves as GEMM
//        operands as well
struct CgStep {
  float* q; float* r; const float* d; const float* Hd; size_t n;
  const double* dHd; int n_dHd; const double* rs_partial; int n_rs; float* rs; double* partials;
  const float* lam; const float* w; float* out;
};
struct CgDirJob { const float* r; float* d; int rows, cols; void* out; int ld; void* outT; int ldT; const float* br; float* bd; };
struct CgDirBatch { int n = 0; int block_begin[MAX_PROBLEMS + 1]; CgDirJob j[MAX_PROBLEMS]; const double* partials; int n_partial; const float* rs; float* rs_new; };
int launch_cg_step(Ctx&, const CgStep&);       // returns the number of partial sums
// Both at once for up to CG_ONE parameters: every workgroup forms all of the new residual for <r, r>; the residual goes to
// another place, since others are still reading it.  at, bias: offsets into the flat vectors (bias -1: none)
constexpr size_t CG_ONE = 16384;
struct CgUpdateJob { long long at, bias; int rows, cols; void* out; int ld; void* outT; int ldT; };
struct CgUpdate {
  int n = 0; int block_begin[MAX_PROBLEMS + 1]; CgUpdateJob j[MAX_PROBLEMS];
  float* q; const float* r; float* r_out; float* d; const float* Hd; int params;
  const double* dHd; int n_dHd; const double* rs_partial; int n_rs; const float* rs; float* rs_new;
};
void launch_cg_update(Ctx&, Elem, CgUpdate&);
void launch_cg_dir(Ctx&, Elem, CgDirBatch&);
void launch_adam(Ctx&, float* x, const float* g, float* m, float* v, float lr, float beta1, float beta2, float eps,
                 float bias1, float bias2, size_t n);
// sum_i s_i ell_i (+ the sum of n partial)
void launch_weighted_loss_sum(Ctx&, const float* s, const float* ell, int rows, const double* partial, int n, float* out);
void launch_label_noise(Ctx&, const int32_t* y, const uint32_t* words, const int32_t* alt,
                        unsigned long long threshold, int n, int32_t* y_out, uint8_t* mask);

// ---- narrow.hip : all layers of a few samples in one workgroup ----------------------------------------
// Everything per layer l = 1 .. L is indexed by l - 1 (weights and what leaves layer l); operands as in the workspace.
constexpr int NARROW_MAX_L = 8, NARROW_ROWS = 16;
struct NarrowSplit { int ks, per, by_nt; };            // K groups, steps of each; multiplier for division by the tiles (narrow_splits)
struct NarrowNet {
  int L, first;                       // the first layer the kernel does itself: 1, or 2 with a_1 (R a_1) formed before
  int n[NARROW_MAX_L + 1], np[NARROW_MAX_L + 1];       // widths, padded
  NarrowSplit fwd[NARROW_MAX_L], bwd[NARROW_MAX_L];
  int act, loss, pitch, ldz;          // elements between rows of the LDS operands; floats between rows of the logits
};
// First-order pass: activations, loss, deltas
struct NarrowGradSide {
  const void* X;                      // operand type of the forward products
  const void* A1;                     // ... as is a_1 where first = 2
  const void* Wf[NARROW_MAX_L];       // W_l^T for the forward products
  const void* Wn[NARROW_MAX_L];       // W_l for the backward products
  const float* bias[NARROW_MAX_L];    // or null
  void* A[NARROW_MAX_L]; void* At[NARROW_MAX_L]; void* D[NARROW_MAX_L]; void* Dt[NARROW_MAX_L];   // (D null for layer 1)
  float* dphi[NARROW_MAX_L]; float* e2[NARROW_MAX_L];                                               // (e2 null: not asked for)
  const Labels* labels; const float* omega_fixed;
  float* ZL; float* P; float* ell; float* s; float* omega; float* dsig;
  int B, Bp, reweight; float inv_batch;
};
struct NarrowGradArgs { NarrowNet net; NarrowGradSide side[2]; int blocks0; const float* theta; int hidden; };
// Forward-over-reverse pass: R-forward, loss Hessian, R-backward; or (cvec) R-forward and <dl_i/dz, Rz_L,i>
struct NarrowRopArgs {
  NarrowNet net;
  const void* X; const void* RA1;     // (RA1: R a_1 where first = 2)
  const void* Wt[NARROW_MAX_L]; const void* Vt[NARROW_MAX_L]; const void* Wn[NARROW_MAX_L]; const void* Vn[NARROW_MAX_L];
  const float* cbias[NARROW_MAX_L];
  const void* A[NARROW_MAX_L]; const void* D[NARROW_MAX_L];
  const float* dphi[NARROW_MAX_L]; const float* e2[NARROW_MAX_L]; float* Rz[NARROW_MAX_L];
  void* RAt[NARROW_MAX_L]; void* RDt[NARROW_MAX_L];
  const float* P; const float* s; const float* Z; const Labels* labels; float* cvec;
  int B, Bp;
};
// The same pass with the weights of all links in LDS from the start (staged_rop_kernel).  Places in LDS are bytes, -1: absent.
constexpr int STAGED_PARTS = 2 * NARROW_MAX_L, STAGED_UNITS = 128;
// products that do not wait for the chain: 16-tiles of A W^T
struct StagedPart {
  const void* A[2]; const void* W[2]; // rows of ld elements; one product, or the sum of two
  const float* bias;                  // or null
  const float* dphi; const float* e2; const float* Rz;    // of the layer whose quantity leaves (some address where not used)
  int ld, steps, N, ldf;
  int products, S, D, E;              // where the sums, phi' and phi'' go
  int finish;                         // what S is: 0 the sum (+ bias), 1 sum phi', 2 sum phi' + phi'' Rz
};
struct StagedWeights { const void* src; int ld, rows, cpr; unsigned inv; int group0; };   // cpr: 16-byte chunks a row, one of them room between rows; inv: 2^32 / cpr
struct StagedLink { void* outT; int w, wpitch, steps, N, F, D, T, E; };        // weights in LDS, summand, phi', what the backward link adds, phi''
struct StagedArgs {
  unsigned short unit[STAGED_UNITS];  // part and 16-tile (<< 4) of a unit
  int units, groups, n_w, n_fwd, n_bwd;
  int B, Bp, C, pitch, buf, zl, ldz, loss, ldp;
  const float* P; const float* s; const float* Z; const Labels* labels; float* cvec; void* RDt;
  StagedWeights w[STAGED_PARTS];      // those of the forward links, then of the backward links, in groups of 64 chunks
  StagedPart part[STAGED_PARTS];
  StagedLink fwd[NARROW_MAX_L], bwd[NARROW_MAX_L];
  int bytes;                          // of LDS
};
static_assert(sizeof(StagedArgs) <= 3840, "passed by value as kernel arguments");
// false: it does not fit (which does not depend on the pointers)
bool staged_plan(const NarrowRopArgs&, Elem, bool curvature, StagedArgs&);
void launch_staged_rop(Ctx&, Elem, bool curvature, const StagedArgs&, double flops);
static_assert(sizeof(NarrowGradArgs) <= 3072 && sizeof(NarrowRopArgs) <= 3072, "passed by value as kernel arguments");
// LDS of a workgroup, and the padded row of its operands; `wide`: the forward operands are fp32
size_t narrow_lds(NarrowNet&, Elem, bool wide);
void launch_narrow_grad(Ctx&, Elem, bool wide, NarrowGradArgs&, int n_sides, double flops);
void launch_narrow_rop(Ctx&, Elem, NarrowRopArgs&, double flops);

// ---- linear.hip : a whole hypergradient of a small single-layer model in one workgroup ----------------
struct LinearArgs {
  const float* X[2]; const float* XT[2]; int ldx, ldxt[2];     // train, validation: fp32 operands [B][ldx], [n_in][ldxt]
  const Labels* labels;                                         // [2]
  int B[2], n_in, C, bias, loss, K;
  float alpha;                                                  // (Neumann)
  const float* w; const float* lam; float* out;
  float* G;                                                     // squared error: room for X^T X (linear_gram_bytes), or null
};
bool linear_fits(int n, int C, int B, int Bv, bool mse, bool cg);   // n: features and bias
size_t linear_gram_bytes(int n);
void launch_linear_hypergrad(Ctx&, const LinearArgs&, bool cg);

}  // namespace betty
