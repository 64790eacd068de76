// Host side of libbetty_hip.so: handle, argument validation, workspace plan, and the launch
// sequences of the five hot-path calls (paper Sec. 3.2; Neumann and finite-difference
// approximate implicit differentiation followed by the mixed second-order VJP).
#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <new>
#include <cstring>
#include <mutex>

#include "internal.h"

using namespace betty;

namespace betty {

void Ctx::begin(int kind, double flops, double bytes) {
  ++launches;
  if (!profiling) return;
  ProfRec r{};
  r.kind = kind; r.flops = flops; r.bytes = bytes; r.ms = -1.f;
  if (hipEventCreate(&r.e0) != hipSuccess || hipEventCreate(&r.e1) != hipSuccess) { profiling = false; return; }
  (void)hipEventRecord(r.e0, stream);
  recs.push_back(r);
}

void Ctx::end() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess && first_error == hipSuccess) first_error = e;
  if (profiling && !recs.empty()) (void)hipEventRecord(recs.back().e1, stream);
}

}  // namespace betty

namespace {

struct LayerInfo {
  int n_in, n_out, n_in_p, n_out_p;
  size_t w_off, b_off;       // offsets (in floats) into a flat parameter vector
};

// Buffers that depend on which batch (train / validation) is being propagated.
struct SideBuf {
  int B = 0, Bp = 0;
  size_t X = 0, XT = 0;                       // a_0 and its transpose
  std::vector<size_t> A, At, D, Dt;           // a_l (1..L-1), delta_l (1..L), each in both orientations
  std::vector<size_t> dphi, e2;               // fp32 phi'(z_l); phi''(z_l) then (delta W^T) phi''
  size_t ZL = 0, P = 0, ell = 0, s = 0, omega = 0, dsig = 0;   // dsig: omega (1 - omega)
  size_t ell_bar = 0, omega_bar = 0, dsig_bar = 0;   // frozen per-sample values (finite differences, reweighting)
};

// One complete set of GEMM operands in a given element type.
struct OperandSet {
  Elem elem = ELEM_F32;
  bool present = false;
  SideBuf side[2];                            // 0 = train (lower), 1 = validation (upper)
  std::vector<size_t> Wn, Wt, Vn, Vt;         // W_l as stored / transposed; same for the direction
  std::vector<size_t> Vn2, Vt2;               // second set of direction copies (pipelined recurrence; main set only)
  std::vector<size_t> RA, RAt, RD, RDt, Rz;   // R-op quantities (train side only)
  size_t cvec = 0;
  // The Neumann series in sample space (main set of the costs without a per-parameter diagonal).  Per layer,
  // over pairs of train samples: G = a a^T (+ 1 for the bias), E = delta delta^T, M = a Ra^T, N = delta R delta^T,
  // and against the validation samples Gx, Ex; all as A operands (EPI_GRAM).  AS = a V + c and DS = delta V^T
  // (fp32) for the current partial sum, Ag and Dg for the vector the series is applied to; the sums of
  // R a and R delta over the steps (proximal cost).
  bool samples = false;
  int ldG = 0, ldGx = 0;
  std::vector<size_t> G, E, M, N, Gx, Ex, AS, DS, Ag, Dg, sumRA, sumRD;
  size_t RA1 = 0, RA1t = 0;   // second place for R a_1, which a step's update writes while it is still being read
};

}  // namespace

namespace {
struct Pass;
// Which form the forward-over-reverse pass takes (main operand set): 0 = launches, or the first layer of narrow.hip's kernels;
// microseconds that a pass is shorter than by launches
struct NarrowForm { int first = 0; bool staged = false; double saving = 0.0; };
}

struct betty_handle_s {
  betty_problem_desc desc{};
  std::vector<int> dims;
  std::vector<LayerInfo> layers;
  int L = 0;
  size_t d = 0, n_hyper = 0;
  int max_np = 0, max_Bp = 0;
  std::string err;
  Ctx ctx;
  char* ws = nullptr;
  size_t ws_need = 0;
  size_t ws_product = 0;     // ... of which a stand-alone product needs no more than this (what only the series and the sums use comes last)
  bool bound = false, batches = false;
  unsigned long long epoch = 0;   // process-wide unique stamp of the last betty_bind
  OperandSet sets[2];        // [0]: element type of desc.prec; [1]: fp32 set for finite differences when prec is bf16
  OperandSet fd_minus;       // fp32, train side only: the evaluation at w - eps v, which runs beside the one at w + eps v
  size_t vec_g = 0, vec_v = 0, vec_p = 0, vec_Hv = 0;
  size_t vec_r = 0;          // second place of the residual (cg_update_kernel)
  size_t bias_pm[2] = {0, 0};        // biases of the two perturbed points (flat layout; only the bias slices are used)
  size_t partials = 0, scalars = 0;
  size_t fd_z1 = 0;          // z_1 of the train batch at w (finite differences)
  size_t sums = 0;           // what the weight-gradient launches sum up beside their results (Epilogue::partial)
  size_t labels = 0;         // Labels[2]: train, validation
  size_t lin_gram = 0;       // (linear.hip)
  size_t logrho = 0;         // proximal cost: log(rho_j) per parameter (a large negative value where rho_j = 0)
  // A hypergradient call repeated with the same arguments is replayed from a captured HIP graph.  Each kind of call
  // keeps the graphs of its last few argument sets: results that a caller lets the allocator place
  // alternate between a few addresses.
  // Steps, gradients and single products are launched directly: the host keeps ahead of the chip (momentum-SGD
  // step of 1024-512-512-10 at batch 256: 42.3 us, replayed 46.8), and recording costs as much as a call takes (a
  // new learning rate every second step of 64-32-4: 33.6 us a step recorded, 16.5 direct).  Only where they are
  // many launches of a small model does the host fall behind.  60 models, direct over replayed: up to 7 launches
  // 0.82 ... 0.97; from 10 and up to 100 000 parameters 0.96 ... 1.29 (alone 1.3 ... 1.6), up to 340 000 1.02 (alone
  // 1.2); more parameters 0.93 ... 0.99 (alone 1.0).
  // They are recorded at the third call with the same arguments, and twice as late each time a recording made way
  // for another before it was replayed 16 times (recording costs 12 to 70 us, a replay saves 1 to 25).
  struct CallKey {
    const void* ptr[6] = {};
    int k[2] = {-1, -1};
    float f[4] = {};
    unsigned long long other_epoch = 0;       // the three-level chain: the binding of its other handle
    bool operator==(const CallKey& o) const {
      return !memcmp(ptr, o.ptr, sizeof ptr) && !memcmp(k, o.k, sizeof k) && !memcmp(f, o.f, sizeof f) && other_epoch == o.other_epoch;
    }
  };
  struct GraphSlot {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    CallKey key;
    unsigned long long used = 0;              // 0: empty
    unsigned long long launches = 0;          // of the first, direct call
    int calls = 0, replays = 0;
  };
  enum { CALL_NEUMANN, CALL_FD, CALL_CG, CALL_BEST_RESPONSE, CALL_CHAIN,
         CALL_SHORT, CALL_HVP = CALL_SHORT, CALL_LOWER, CALL_UPPER, CALL_MIXED, CALL_SGD, CALL_KINDS };
  static constexpr int SHORT_LAUNCHES = 10;
  static constexpr size_t SHORT_PARAMS = 350000;
  int record_after[CALL_KINDS - CALL_SHORT] = {2, 2, 2, 2, 2};   // direct calls before a short kind is recorded
  static constexpr int SLOTS = 4;
  GraphSlot graphs[CALL_KINDS][SLOTS];
  unsigned long long graph_clock = 0;
  hipStream_t capture_stream = nullptr;       // sequences are recorded here and replayed on ctx.stream
  hipStream_t bound_stream = nullptr;         // betty_bind; ctx.stream is where the calls run (betty_run_on)
  hipEvent_t order_event = nullptr;
  bool use_graphs = true;
  int tune_tile128_min = 512;                 // see plan_chain (measured on 512x4096x8192: 64-tiles beat 128-tiles until the grid is several waves deep)
  bool tune_split = true, tune_rect_forced = false;   // K-split kernels allowed; 128 x 64 tiles for everything unsplit
  int tune_wgrad_cfg = GEMM_64x1;
  int tune_wgrad128_min = 512;                // 128-tiles a bf16 weight-gradient launch needs to use the 128-tile kernel (0 = never, and 64-tiles for every launch)
  // For large models the Neumann recurrence overlaps each layer's weight-gradient launch
  // (bandwidth-bound) with the rest of the R-backward chain on a second stream of the same
  // priority.  Every cross-stream dependency costs several microseconds (measured: 5 per product,
  // about 37 us in total), so it only pays when the launches it hides are far longer than that:
  // it is switched on from 32M parameters (+1 % at 116M parameters, -25 % at 5M).
  hipStream_t side_stream = nullptr;
  std::vector<hipEvent_t> fork_events;        // one per layer
  hipEvent_t join_event = nullptr;
  bool use_pipeline = false;
  // Optimiser steps with bf16 operands keep one grouping of the sums along K, whatever kernel the launch
  // rule picks elsewhere: activations and deltas are rounded to bf16 after every layer, so another grouping
  // sends a training run down another trajectory (up to 3e-3 in the momentum after a step or three).  What
  // the rule would save is small but for ragged models: a step of 3072-1024-1024-1024-10 at batch 256 72.6 / 72.5 us,
  // 1024-512-512-10 36.9 / 35.6, 2048-2048-2048-1000 at 512 181 / 173, 777-301-65-33 at 130 48.3 / 35.3.
  bool fixed_grouping = false;
  NarrowForm rop_form;
  const Pass* z1_pass = nullptr;       // first-order passes leave z_1 of this pass in fd_z1
  bool layer1_done = false;                   // a_1 and phi'(z_1) of the passes are there already (finite differences)
  bool as_pair = false;                       // choose kernels for single passes as if two shared the launch
  bool tune_pair_forced = false;              // 64-tiles with a two-way K split for every activation-shaped product
  int tune_narrow = -1;                       // narrow.hip: 0 never, 1 or 2 that first layer wherever it fits, -1 by size
  int tune_linear = -1;                       // one-workgroup kernel for single-layer models: 0 never, 1 wherever it fits, -1 by size
  int tune_layer1 = -1;                       // finite differences, layer 1 of both points from one product: 0 never, 1 wherever it can be, -1 by size
  int tune_samples = -1;                      // sample-space series: 0 never, 1 wherever it exists, -1 by size
  // Finite differences: the passes at w + eps v and w - eps v share their launches, with weight operands
  // for both points; above 32M parameters, where either alone fills the chip, they follow each other on one
  // set of weight operands.  Same kernels on the same data: not a bit differs.
  bool fd_paired = false;

  template <typename T = void> T* at(size_t off) const { return (T*)(ws + off); }
  float* f(size_t off) const { return (float*)(ws + off); }
};

namespace {

betty_status fail(betty_handle h, betty_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (h) h->err = buf;
  return st;
}

struct Planner {
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return o;
  }
};

// Extent of a launch: output tiles of each size over all its problems, and the 64-byte steps along K
// of the longest one.
struct Extent {
  long t16 = 0, t32 = 0, t64 = 0, t128 = 0, rect = 0;
  int steps = 0;
  static long up(int n, int t) { return (n + t - 1) / t; }
  void add(Elem elem, int M, int N, int K0, int K1) {
    const int per = 64 / (int)elem_size(elem);
    t16 += up(M, 16) * up(N, 16);
    t32 += up(M, 32) * up(N, 32);
    t64 += up(M, 64) * up(N, 64);
    rect += up(M, 128) * up(N, 64);
    t128 += up(M, 128) * up(N, 128);
    steps = std::max(steps, (int)(up(K0, per) + up(K1, per)));
  }
};

void plan_side(betty_handle h, Planner& pl, SideBuf& sb, Elem elem, int B, bool curvature, bool inputs = true) {
  const int L = h->L;
  const size_t es = elem_size(elem);
  sb.B = B;
  sb.Bp = padup(B);
  const size_t Bp = sb.Bp;
  if (inputs) {
    sb.X = pl.take(Bp * h->layers[0].n_in_p * es);
    sb.XT = pl.take((size_t)h->layers[0].n_in_p * Bp * es);
  }
  sb.A.assign(L + 1, 0); sb.At.assign(L + 1, 0); sb.D.assign(L + 1, 0); sb.Dt.assign(L + 1, 0);
  sb.dphi.assign(L + 1, 0); sb.e2.assign(L + 1, 0);
  for (int l = 1; l <= L; ++l) {
    const size_t np = h->layers[l - 1].n_out_p;
    if (l < L) {
      sb.A[l] = pl.take(Bp * np * es);
      sb.At[l] = pl.take(np * Bp * es);
      sb.dphi[l] = pl.take(Bp * np * 4);
      if (curvature && h->desc.act == BETTY_ACT_GELU_ERF) sb.e2[l] = pl.take(Bp * np * 4);
    }
    sb.D[l] = pl.take(Bp * np * es);
    sb.Dt[l] = pl.take(np * Bp * es);
  }
  const size_t Cp = h->layers[L - 1].n_out_p;
  sb.ZL = pl.take(Bp * Cp * 4);
  sb.P = pl.take(Bp * Cp * 4);
  sb.ell = pl.take(Bp * 4);
  sb.s = pl.take(Bp * 4);
  sb.omega = pl.take(Bp * 4);
  sb.ell_bar = pl.take(Bp * 4);
  sb.omega_bar = pl.take(Bp * 4);
  sb.dsig = pl.take(Bp * 4);
  sb.dsig_bar = pl.take(Bp * 4);
}

// How much of an operand set exists:
//  SET_FULL          everything (first-order passes on both batches and the forward-over-reverse passes)
//  SET_FIRST_ORDER   what first-order gradients on both batches touch (the fp32 set that serves the
//                    finite-difference variant and the fp32 forward of ReLU networks beside bf16 operands)
//  SET_TRAIN_ONLY    just what a gradient of the lower cost on the train batch touches
//  SET_ACTIVATIONS   the same without weight operands
enum SetScope { SET_FULL, SET_FIRST_ORDER, SET_TRAIN_ONLY, SET_ACTIVATIONS };

void plan_set(betty_handle h, Planner& pl, OperandSet& os, Elem elem, bool second_direction_set, SetScope scope) {
  const int L = h->L;
  const size_t es = elem_size(elem);
  os.elem = elem;
  os.present = true;
  const bool inputs = scope == SET_FULL || scope == SET_FIRST_ORDER;
  plan_side(h, pl, os.side[0], elem, h->desc.batch_train, scope == SET_FULL, inputs);
  if (scope == SET_ACTIVATIONS) return;
  os.Wn.assign(L, 0); os.Wt.assign(L, 0); os.Vn.assign(L, 0); os.Vt.assign(L, 0);
  for (int i = 0; i < L; ++i) {
    const size_t m = (size_t)h->layers[i].n_in_p * h->layers[i].n_out_p * es;
    os.Wn[i] = pl.take(m); os.Wt[i] = pl.take(m);
    if (scope == SET_FULL) { os.Vn[i] = pl.take(m); os.Vt[i] = pl.take(m); }
  }
  if (scope == SET_TRAIN_ONLY) return;
  plan_side(h, pl, os.side[1], elem, h->desc.batch_val, false);
  const size_t Bp = os.side[0].Bp;
  os.cvec = pl.take(Bp * 4);
  if (scope == SET_FIRST_ORDER) return;
  if (second_direction_set) {
    os.Vn2.assign(L, 0); os.Vt2.assign(L, 0);
    for (int i = 0; i < L; ++i) {
      const size_t m = (size_t)h->layers[i].n_in_p * h->layers[i].n_out_p * es;
      os.Vn2[i] = pl.take(m); os.Vt2[i] = pl.take(m);
    }
  }
  os.RA.assign(L + 1, 0); os.RAt.assign(L + 1, 0); os.RD.assign(L + 1, 0); os.RDt.assign(L + 1, 0);
  os.Rz.assign(L + 1, 0);
  for (int l = 1; l <= L; ++l) {
    const size_t np = h->layers[l - 1].n_out_p;
    if (l < L) { os.RA[l] = pl.take(Bp * np * es); os.RAt[l] = pl.take(np * Bp * es); }
    os.RD[l] = pl.take(Bp * np * es);
    os.RDt[l] = pl.take(np * Bp * es);
    os.Rz[l] = pl.take(Bp * np * 4);
  }
}

// Microseconds by which the Neumann series in sample space (neumann_samples_seq) is faster than the
// parameter-sized recurrence in a call of K steps, from the validation gradient or from a dense vector: the
// operations of either form, the traffic of parameter-sized vectors and of matrices over pairs of samples, what
// launches cost beyond that (a single layer's link is a long reduction over few tiles: its share goes with n_in), and
// the proximal cost's weighted sums (a launch a step but the last).  The constants are a fit to 12 000 calls timed in
// both forms: 600 models of one to eight layers, widths 13 ... 4096, both costs and element types, batch 32 ... 1024
// against 32 ... 16 384 validation samples, K = 1 ... 15.  The choice is 0.5 % behind the better form on average and
// beats parameters alone by 7 %; a step's share taken by itself, without what begins a call, was 3 % behind (and up
// to three times slower: 256-128-128-10, 16 384 validation samples, K = 1: 217 us on parameters, 358 us in sample space).
double samples_saving(betty_handle h, int K, bool dense) {
  const bool bf16 = h->desc.prec == BETTY_PREC_BF16_FP32ACC, prox = h->desc.hp == BETTY_HP_PROXIMAL, one = h->L == 1;
  const double B = h->desc.batch_train, Bv = h->desc.batch_val, per_pair = bf16 ? 10.0 : 6.0, split = bf16 ? 2.0 : 1.0;
  // microseconds an operation: links, updates through the pair matrices, the pair matrices themselves, validation side
  const double t_link = bf16 ? 0.9e-9 : 7.5e-9, t_pair = bf16 ? 1.3e-9 : 4.5e-9, t_gram = bf16 ? 0.0 : 8.5e-9;
  const double t_begin = bf16 ? 1.4e-9 : 8.5e-9, t_val = bf16 ? 1.1e-9 : 8.5e-9;
  // ... a parameter, in a step and in the first gradient; one pass over the pairs of train samples, a pair with a validation sample
  const double t_param = bf16 ? 5.5e-6 : 6e-6, t_first = bf16 ? 5.5e-6 : 9e-6;
  const double pairs = (bf16 ? 1.2e-6 : 2e-6) * B * B, t_cross = 2.4e-6;
  const double long_sum = (bf16 ? 2e-3 : 4.5e-3) * h->layers[0].n_in;
  double step = bf16 ? 2.0 : one ? 3.0 : 4.5, begin = 3.5, sums = 4.7;
  if (one) { step += long_sum; begin += long_sum; }
  for (int i = 0; i < h->L; ++i) {
    const double n_in = h->layers[i].n_in, n_out = h->layers[i].n_out, up = i == 0 ? 0.0 : 1.0;
    step += (4.0 + 4.0 * up) * B * n_in * n_out * t_link + n_in * n_out * t_param;
    step -= (i == 0 ? (per_pair - 4.0) * n_out : per_pair * (n_in + n_out)) * B * B * t_pair;
    step -= (1.0 + 5.0 * up) * pairs;                    // G, E read, M, N written and read
    sums += 10e-6 * B * n_out;
    if (K > 0) begin += 2.0 * B * B * (n_in + up * n_out) * t_gram + (1.0 + up) * pairs;
    if (dense) {
      begin += (2.0 + 2.0 * up) * B * n_in * n_out * t_begin;
    } else {
      begin += 2.0 * B * Bv * (n_in + up * n_out + split * (n_out + up * n_in)) * t_begin + (1.0 + up) * B * Bv * t_cross;
      if (!prox) begin -= 2.0 * Bv * n_in * n_out * t_val + n_in * n_out * t_first;   // (the proximal cost forms that gradient in either case)
    }
  }
  return K * step - begin - (prox && K > 1 ? (K - 1) * sums : 0.0);
}
// Models with narrow layers take all layers of a few samples in one workgroup (narrow.hip).  Whether the first-order
// passes over that many samples together (rop = false) or the forward-over-reverse pass does, and from which layer on: 0 =
// launches per layer, 1, or 2 = layer 1, whose reduction may be long, stays a launch of its own.
// By the estimated time: a launch taken as 4.7 us whatever its width (up to about 256; now nearer 4, but a lower price leaves more of the fused
// form's gain than it saves), the fused kernel 6 us, 1.6 us a link, and 1 us per 9 KB of weights: that is the latency of fetching them link by link
// in every workgroup, far below what a compute unit can read.  Chosen forms over launches, up to 4096 samples: first-order passes of 500 models
// 17.8 ms in all, 17.3 with the better form of each, 21.0 by launches, 2 more than 3 % slower, up to 1.11 times; forward-over-reverse passes beside
// the form in LDS below (choose_rop_form).
// Beyond, workgroups share compute units and the launches fill the chip, soonest where the output is wide (a narrow one has
// kernels of its own that cost the launches more).  Fused over launches, 400 models of each kind of pass: forward-over-reverse with more than 16
// outputs 0.91 up to 8192 samples, 1.05 ... 1.6 beyond; up to 16 outputs, bf16 0.91 up to 8192, 0.99 ... 1.04 up to 12288, 1.1 ... 1.25 beyond, fp32
// 0.91 ... 0.94 up to 8192, 0.96 ... 1.03 up to 24576, 1.07 beyond.  First-order with more than 16 outputs 0.64 ... 0.95 up to 32768, 1.05 beyond;
// up to 16 outputs 0.70 ... 0.94 up to 66000, 1.13 times at most.
// (Forward-over-reverse passes: 32-wide, 8 layers 66 us by launches, 29 us; 64-wide fp32, 4 layers 28 / 23 us; 128-wide 28 / 47 us, with
// bf16 operands 28 / 32 us.)
int narrow_max_samples(betty_handle h, bool rop, Elem elem) {
  if (h->dims[h->L] > LAST_ROP_MAX_C) return rop ? 4096 : 24576;
  return !rop ? INT_MAX : elem == ELEM_BF16 ? 12288 : 32768;
}
int launches_per_layer(betty_handle h, bool rop) {
  return 2 * h->L - (h->dims[h->L] <= LAST_ROP_MAX_C ? 2 : rop && h->dims[h->L] <= 32 ? 1 : 0);
}
struct NarrowEstimate { double fused, launches; int first; };
NarrowEstimate narrow_estimate(betty_handle h, bool rop, Elem elem) {
  const int L = h->L;
  const bool bf16 = elem == ELEM_BF16;
  const double launch = 4.7, per_kb = 1.0 / 9, es = bf16 ? 2.0 : 4.0, fwd_es = !rop && bf16 && h->desc.act == BETTY_ACT_RELU ? 4.0 : es;
  const double launches = launch * launches_per_layer(h, rop), pairs = rop ? 2.0 : 1.0;
  double fused = 6.0, first_link = 0;
  for (int l = 1; l <= L; ++l) {
    const double kb = (double)h->dims[l - 1] * h->dims[l] / 1024.0;
    const double forward = 1.6 + (l > 1 ? pairs : 1.0) * kb * fwd_es * per_kb;
    if (l == 1) first_link = forward;
    fused += forward + (l > 1 ? 1.6 + pairs * kb * es * per_kb : 0.0);
  }
  const bool split = L >= 3 && launch < first_link;
  return NarrowEstimate{split ? fused - first_link + launch : fused, launches, split ? 2 : 1};
}
int narrow_first(betty_handle h, bool rop, Elem elem, int samples) {
  const int L = h->L;
  if (L < 2 || L > NARROW_MAX_L || h->tune_narrow == 0) return 0;
  NarrowNet net{};
  net.L = L;
  for (int l = 0; l <= L; ++l) net.n[l] = h->dims[l];
  if (narrow_lds(net, elem, elem == ELEM_BF16) > 150 * 1024) return 0;
  if (h->tune_narrow > 2) return 0;
  if (h->tune_narrow > 0) return L >= 3 ? h->tune_narrow : 1;
  const NarrowEstimate e = narrow_estimate(h, rop, elem);
  return samples <= narrow_max_samples(h, rop, elem) && e.fused < 0.92 * e.launches ? e.first : 0;
}
NarrowNet narrow_net(betty_handle h, int first);
// The forward-over-reverse pass with all weights in LDS (staged_rop_kernel), from layer `first` on: its estimated time, or
// infinity where it does not fit (which does not depend on the pointers).  4 us, 0.6 us a link, the products with operands of the
// direction alone by the steps of a wavefront (bf16 0.75 us, fp32 1 us) and those that one 16-tile makes one after the other beyond
// four, 0.04 us a KB of weights, 3.3 us for layer 1 by itself.
double staged_estimate(betty_handle h, Elem elem, int first) {
  if (h->L < 2 || h->L > NARROW_MAX_L || first > (h->L >= 3 ? 2 : 1)) return INFINITY;
  NarrowRopArgs r{};
  StagedArgs a;
  r.net = narrow_net(h, first);
  narrow_lds(r.net, elem, false);
  if (!staged_plan(r, elem, h->desc.act == BETTY_ACT_GELU_ERF, a)) return INFINITY;
  int steps = 0, longest = 0;
  for (int u = 0; u < a.units; ++u) {
    const StagedPart& p = a.part[a.unit[u] & 15];
    const int n = p.steps * p.products;
    steps += n;
    longest = std::max(longest, n);
  }
  return 4.0 + 0.6 * (a.n_fwd + a.n_bwd) + (elem == ELEM_BF16 ? 0.75 : 1.0) * steps / 16 + 0.2 * std::max(0, longest - 4) + 0.04 * a.groups +
         (first > 1 ? 3.3 : 0.0);
}
// The form of the forward-over-reverse pass: the one in LDS where it takes less than 0.94 of 4.0 us a launch.  Steps of the series of
// 1500 models (2 to 8 layers, up to 320 wide, 8 to 1500 inputs, batch 16 to 3000): 40.4 ms by the rule, 40.1 with the better form of each, 53.1 by
// launches; 11 of them more than 3 % slower than launches, one 1.18 times, the others up to 1.13.  Up to 4096 samples: a workgroup has a
// compute unit's LDS to itself.
// What it saves beside the series over samples, whose estimate counts launches: 3.2 us a launch, those of up to 32 outputs 2 or 3 us more.  Calls of
// 2600 reweighting and proximal models: 0.25 % behind the better of samples and parameters, 8 of those that take this pass more than 3 %, up to
// 1.09 times (at 4.7 us a launch 21 of them, up to 1.4 times: 511-12-34, batch 50, fp32, K = 9 127 us, on parameters 181).
NarrowForm choose_rop_form(betty_handle h, Elem elem) {
  const int C = h->dims[h->L];
  const double n = launches_per_layer(h, true);
  const double one = h->tune_narrow >= 0 && h->tune_narrow < 3 ? INFINITY : staged_estimate(h, elem, 1);
  const double two = h->tune_narrow >= 0 && h->tune_narrow < 3 ? INFINITY : staged_estimate(h, elem, 2);
  const double time = std::min(one, two), gain = 4.0 * n - time;
  const NarrowForm staged{two < one ? 2 : 1, true, std::max(0.0, 3.2 * n + (C <= LAST_ROP_MAX_C ? 3.0 : C <= 32 ? 2.0 : 0.0) - time)};
  if (h->tune_narrow >= 3) {
    if (h->L >= 3 && h->tune_narrow == 4) return std::isfinite(two) ? NarrowForm{2, true, 0.0} : NarrowForm{};
    return std::isfinite(one) ? NarrowForm{1, true, 0.0} : NarrowForm{};
  }
  NarrowForm f{narrow_first(h, true, elem, h->desc.batch_train), false, 0.0};
  // Half of the estimate less 2 us: it is 0.8 of it on average, nothing with two layers or few rows, and the saving in sample space
  // is underestimated where this is.  (371 models with narrow layers, series of 1, 3 and 9 steps over launches only: 0.800, the
  // better form of every call 0.798, 9 of 2226 calls more than 3 % slower; narrow layers always: up to 1.26, 915-33-33-146,
  // batch 25, K = 9 208 -> 264 us.)
  const NarrowEstimate e = narrow_estimate(h, true, elem);
  if (f.first) f.saving = std::max(0.0, 0.5 * (e.launches - e.fused) - 2.0);
  return h->desc.batch_train <= 4096 && gain > std::max(0.06 * 4.0 * n, f.saving) ? staged : f;
}
int narrow_rop_first(betty_handle h) { return h->rop_form.first; }

// What the fused pass takes off a step of the recurrence over parameters, which samples_saving counts by launches
double narrow_saving(betty_handle h) { return h->rop_form.saving; }

bool has_samples_form(betty_handle h, int K) { return h->desc.hp == BETTY_HP_REWEIGHT_NET || (h->desc.hp == BETTY_HP_PROXIMAL && K > 0); }

bool use_samples(betty_handle h, int K, bool dense) {
  return h->sets[0].samples && has_samples_form(h, K) && (h->tune_samples == 1 || samples_saving(h, K, dense) > K * narrow_saving(h));
}

// Whether any call with steps takes that form (both estimates are linear in K beyond 1).
bool plans_samples(betty_handle h) {
  if (h->tune_samples >= 0) return h->tune_samples == 1 && has_samples_form(h, 1);
  for (int K : {1, 1 << 20})
    for (bool dense : {false, true})
      if (has_samples_form(h, K) && samples_saving(h, K, dense) > K * narrow_saving(h)) return true;
  return false;
}

// What the series in sample space needs of the main operand set.  The matrices over pairs of samples are
// quadratic in the batch, so they are planned only where the rule above can take that form.
void plan_samples(betty_handle h, Planner& pl, OperandSet& os) {
  const int L = h->L;
  const size_t es = elem_size(os.elem), Bp = os.side[0].Bp;
  os.samples = true;
  const int width = os.elem == ELEM_BF16 ? 2 : 1;           // value and remainder (GemmArgs::split)
  os.ldG = (int)Bp * width;
  os.ldGx = os.side[1].Bp * width;
  for (auto* v : {&os.G, &os.E, &os.M, &os.N, &os.Gx, &os.Ex, &os.AS, &os.DS, &os.Ag, &os.Dg}) v->assign(L + 1, 0);
  for (int l = 1; l <= L; ++l) {
    const size_t np = h->layers[l - 1].n_out_p, ip = h->layers[l - 1].n_in_p;
    os.G[l] = pl.take(Bp * os.ldG * es);
    os.Gx[l] = pl.take(Bp * os.ldGx * es);
    os.AS[l] = pl.take(Bp * np * 4);
    os.Ag[l] = pl.take(Bp * np * 4);
    if (l == 1) continue;
    os.E[l] = pl.take(Bp * os.ldG * es);
    os.M[l] = pl.take(Bp * os.ldG * es);
    os.N[l] = pl.take(Bp * os.ldG * es);
    os.Ex[l] = pl.take(Bp * os.ldGx * es);
    os.DS[l] = pl.take(Bp * ip * 4);
    os.Dg[l] = pl.take(Bp * ip * 4);
  }
  if (L >= 2) {
    const size_t n1 = h->layers[0].n_out_p;
    os.RA1 = pl.take(Bp * n1 * es); os.RA1t = pl.take(n1 * Bp * es);
  }
  if (h->desc.hp != BETTY_HP_PROXIMAL) return;
  os.sumRA.assign(L + 1, 0); os.sumRD.assign(L + 1, 0);
  for (int l = 1; l <= L; ++l) {
    const size_t np = h->layers[l - 1].n_out_p;
    os.sumRD[l] = pl.take(np * Bp * 4);
    if (l < L) os.sumRA[l] = pl.take(np * Bp * 4);
  }
}

// Single-layer models with a decay per parameter and fp32 operands whose data fit one workgroup (linear.hip)
bool has_linear_form(betty_handle h, bool cg) {
  const LayerInfo& li = h->layers[0];
  return h->L == 1 && h->desc.hp == BETTY_HP_L2_DECAY && h->desc.prec == BETTY_PREC_FP32 && h->tune_linear != 0 &&
         linear_fits(li.n_in + (h->desc.has_bias ? 1 : 0), li.n_out, h->desc.batch_train, h->desc.batch_val,
                     h->desc.loss == BETTY_LOSS_MSE, cg);
}

// Whether a call of K steps takes that form, by the estimated microseconds of either.  By launches a call costs little
// more with every output or sample; in one workgroup a product is multiply-adds on four SIMDs (rows, columns: 256
// threads each round), sums over chunks of features that one thread forms per sample and output (chunks), and over
// chunks of samples per parameter (update), each times the outputs, and the beginning costs as much as several steps.  The
// Gram form of the squared error pays for X^T X by the train batch, once, and its steps not at all by it.
// Fitted to 6078 calls timed in both forms (up to 1000 features, 16 outputs, 262144 train samples, K = 0 ... 20): estimates
// within 3 to 4 % (launches) and 6 to 10 % (one workgroup); 26 of the calls that take this form are more than 3 % slower, the worst
// 12 %, and 87 of the others would have been more than 3 % faster, up to 16 % (single steps of squared errors with 10^5
// samples and more 29 %).  (By the number of outputs alone: softmax 401 - 12, batch 64, K = 2
// 36 -> 67 us, conjugate gradient of 64 - 16, batch 512, K = 1 30 -> 57.)  Ridge 64 - 1, batch 512, K = 20: 163 us by
// launches, 16.5 us; softmax 200 - 4, batch 128, K = 5: 52 / 38 us (conjugate gradient 84 / 50).  A step of up to 64 features takes 0.25 us with one
// output, 0.65 with 16, counted as 0.33.  With launches as they are now 674 calls: 0.4 % behind the better form on average, 6 of them more
// than 3 %, at most 11.5 %.
bool use_linear(betty_handle h, bool cg, int K) {
  if (!has_linear_form(h, cg)) return false;
  if (h->tune_linear == 1) return true;
  const LayerInfo& li = h->layers[0];
  if (li.n_out > 16) return false;                          // (as far as it was timed)
  const bool mse = h->desc.loss == BETTY_LOSS_MSE, gram = mse && !cg;
  const int n = li.n_in + (h->desc.has_bias ? 1 : 0), C = li.n_out, train = h->desc.batch_train, val = h->desc.batch_val;
  auto up = [](int x, int m) { return (x + m - 1) / m; };
  const double kn = n * 1e-3, B = train, Bv = val, chunks = up(n, 32);
  const double step = cg ? 11.2 + 5.8 * kn + 2.5e-3 * B + 38e-6 * n * B + 0.07 * C
                         : 4.75 + 3.6 * kn + 3.5e-3 * B + (mse ? 3e-6 : 10e-6) * n * B + 0.02 * C;
  const double launches = (cg ? K == 0 ? 21.3 : 13.2 : 18.6) + (cg ? 2.6 : 4.0) * kn + 3e-3 * Bv + K * step;
  auto rows = [&](int b) { return up(up(n, 32) * up(b, 16) * 16, 256); };
  auto columns = [&](int b) { return up(up(b, 32) * up(n, 16) * 16, 256); };
  auto update = [&](int b) { return up(C * n, 1024) * up(b, 32); };
  double one = (cg ? 7.9 : 7.1) + 1.4 * C * kn;
  one += mse ? C * (0.15 * (rows(val) + columns(val)) + 0.022 * chunks + 0.03) + 0.09 * update(val)
             : C * (0.127 * (rows(val) + columns(val)) + 0.016 * chunks + 0.10) + 0.115 * update(val);
  if (gram) {
    one += K * (n <= 64 ? 0.33 : 0.1 * C * rows(n) + 0.32) - 2.3;
    if (K > 0) one += 2.2 + B * ((train <= 131072 ? 3.3e-3 : 4.2e-3) + 1.57e-5 * 4 * chunks * chunks);
  } else {
    one += K * (C * ((mse ? 0.062 : 0.051) * (rows(train) + columns(train)) + (mse ? 0.02 : 0.025) * chunks + (mse ? 0.14 : 0.26)) + 0.044 * update(train) +
                (cg ? 2.2 : 0.35));
    if (!mse) one += 0.28 * C * rows(train);
  }
  return one < 0.97 * launches;
}

OperandSet& fd_operands(betty_handle h) { return h->sets[1].present ? h->sets[1] : h->sets[0]; }

void plan(betty_handle h) {
  Planner pl;
  const Elem main_elem = h->desc.prec == BETTY_PREC_BF16_FP32ACC ? ELEM_BF16 : ELEM_F32;
  h->rop_form = choose_rop_form(h, main_elem);
  plan_set(h, pl, h->sets[0], main_elem, true, SET_FULL);
  if (main_elem == ELEM_BF16) plan_set(h, pl, h->sets[1], ELEM_F32, false, SET_FIRST_ORDER);
  const size_t vb = h->d * 4;
  h->vec_g = pl.take(vb); h->vec_v = pl.take(vb); h->vec_p = pl.take(vb); h->vec_Hv = pl.take(vb);
  if (h->desc.has_bias) { h->bias_pm[0] = pl.take(vb); h->bias_pm[1] = pl.take(vb); }
  // the second perturbed point of a central difference: activations and deltas of its own, weights of its
  // own where both points go through the same launches
  plan_set(h, pl, h->fd_minus, ELEM_F32, false, h->fd_paired ? SET_TRAIN_ONLY : SET_ACTIVATIONS);
  h->fd_minus.side[0].X = fd_operands(h).side[0].X;      // the same inputs
  h->fd_minus.side[0].XT = fd_operands(h).side[0].XT;
  if (!h->fd_paired) { h->fd_minus.Wn = fd_operands(h).Wn; h->fd_minus.Wt = fd_operands(h).Wt; }
  if (h->desc.hp == BETTY_HP_PROXIMAL) h->logrho = pl.take(vb);
  h->partials = pl.take(1024 * 8);
  h->scalars = pl.take(256);
  h->labels = pl.take(2 * sizeof(Labels));
  h->ws_product = pl.off;
  size_t n_sums = 4096;      // one per finishing wavefront of at most 64-tiles (16-tiles: at most 1024 of them) and per bias
  for (const LayerInfo& li : h->layers) n_sums += 4 * (size_t)Extent::up(li.n_in, 64) * Extent::up(li.n_out, 64) + li.n_out + 4096;
  if (h->L >= 2) h->fd_z1 = pl.take((size_t)h->sets[0].side[0].Bp * h->layers[0].n_out_p * 4);
  h->sums = pl.take(2 * n_sums * sizeof(double));      // (conjugate gradient keeps those of two launches)
  if (h->d <= CG_ONE && h->L <= MAX_PROBLEMS) h->vec_r = pl.take(vb);
  if (plans_samples(h)) plan_samples(h, pl, h->sets[0]);
  if (h->desc.loss == BETTY_LOSS_MSE && has_linear_form(h, false))
    h->lin_gram = pl.take(linear_gram_bytes(h->layers[0].n_in + (h->desc.has_bias ? 1 : 0)));
  h->ws_need = pl.off;
}

// The lower cost's parameter-diagonal term is sum_j exp(c_j) (.)^2 with c = lambda for L2 decay and
// c = log(rho) for the proximal cost; the reweighting cost has none.
const float* diag_log(betty_handle h, const float* lambda) {
  if (h->desc.hp == BETTY_HP_L2_DECAY) return lambda;
  if (h->desc.hp == BETTY_HP_PROXIMAL) return h->f(h->logrho);
  return nullptr;
}
// the weight-net parameters, for the cost that has a weight net
const float* wnet_theta(betty_handle h, const float* lambda) {
  return h->desc.hp == BETTY_HP_REWEIGHT_NET ? lambda : nullptr;
}

// Kernel configuration of an activation-shaped GEMM (M = batch), from its extent.  The lines come from
// timing every configuration on 1 400 shapes (batch 32 ... 1024, widths 8 ... 4096, K 64 ... 8192, both
// element types, one and two problems a launch); the rule stays within 0.6 % of the best on average.  (With 16-tiles
// in whole lines: 710 models, the lines between 16- and 32-tiles moved either way -0.2 ... +1.6 %.)
//  * 16-tiles while every tile has a compute unit of its own (256 of them; bf16 up to 80 steps, where
//    32-tiles with their half as large operand traffic draw level), with short K also beyond:
//    such a launch is bound by latency.  fp32 128 x 256 x 784: 8.9 us on 32-tiles, 6.0 us; bf16
//    130 x 301 x 777: 8.4 us (64-tiles, four-way K split, since removed), 4.6 us;
//  * 32-tiles with an eight-way K split inside the workgroup up to about two and a half per compute
//    unit (bf16 512 x 1024 x 1024: 8.0 us against 10.0 us on 64-tiles; 512 x 2048 x 1024: 12.4 / 10.8);
//  * 128 x 64 tiles (bf16) from about 200 of them, while 64-tiles would come to at most four per compute
//    unit and the reduction is long: such a launch is bound by what a compute unit can pull through its L1
//    (measured: about 63 GB/s each with all of them pulling operands from behind the L2, 88 GB/s out of it), and a 128 x 64 tile fetches 192
//    operand rows for the 8192 outputs that two 64-tiles fetch 256 for (121M-parameter model,
//    batch 512: R-forward link 73 -> 66 us, backward link 76 -> 60 us); with fp32 operands, whose
//    launches of this size are bound by the matrix cores, 64-tiles are 10 % faster;
//  * 64-tiles with a two-way K split (eight wavefronts) while every tile has a compute unit of its own and the
//    reduction is long: four wavefronts leave a SIMD one, with nothing to hide its barriers behind and the whole
//    epilogue to itself (bf16 gradients of 2048-2048-2048-1000 at 512 117 -> 108 us; 40 models -0.3 ... +8 %; with two tiles a
//    compute unit 64-tiles hide each other, and fp32 launches lose up to 5 %);
//  * 128-tiles once there are enough of them to fill the chip several times over (not for layer 1 at both points of a
//    difference, whose epilogue does not fit their registers: 168-812-26 with 23949 samples 1620 -> 2020 us a call);
//  * otherwise plain 64-tiles.
int plan_chain(betty_handle h, Elem elem, GemmBatch& b) {
  if (h->fixed_grouping && elem == ELEM_BF16) {
    // eight, four or one contiguous ranges of 64-element k-tiles of the padded extent; the unsplit kernels
    // all sum in the same order
    long tiles = 0;
    int TT = 0;
    for (int i = 0; i < b.n; ++i) {
      GemmArgs& g = b.p[i].g;
      g.K[0] = padup(g.K[0]);
      tiles += 4L * (padup(g.M) / 128) * (padup(g.N) / 128);
      TT = std::max(TT, g.K[0] / 64);
    }
    if (tiles >= 4L * h->tune_tile128_min) return GEMM_128x1;
    if (tiles <= 128 && TT >= 16) return GEMM_32x8;
    if (tiles < 256 && TT >= 8) return GEMM_32x4;
    return tiles <= 1024 && TT >= 16 ? GEMM_128x64 : GEMM_64x1;
  }
  Extent x;
  for (int r = 0; r < (h->as_pair && b.n == 1 ? 2 : 1); ++r)
    for (int i = 0; i < b.n; ++i) x.add(elem, b.p[i].g.M, b.p[i].g.N, b.p[i].g.K[0], b.p[i].g.K[1]);
  const bool wide_rows = b.p[0].e.mode == EPI_RFWD_LAST_HESS && b.p[0].g.N > 16;   // its row sums need a whole row per tile
  if (h->tune_split && !h->tune_pair_forced && !wide_rows) {
    const int shorter = elem == ELEM_BF16 ? 1 : 2;        // the same K has twice the steps with fp32 operands
    if (x.t16 <= 256 ? (elem == ELEM_F32 || x.steps < 80)
                     : ((x.t16 <= 512 && x.steps <= 12 * shorter) || (x.t16 <= 1024 && x.steps <= 4 * shorter)))
      return GEMM_16;
  }
  if (h->tune_split && !h->tune_pair_forced && x.t32 <= 600) return GEMM_32x8;
  if (!h->tune_pair_forced && x.t128 >= h->tune_tile128_min && b.p[0].e.mode != EPI_FWD_PM) return GEMM_128x1;
  if (h->tune_pair_forced || (h->tune_split && !h->tune_rect_forced && x.t64 <= 256 && x.steps >= 16)) return GEMM_64x2;
  if (h->tune_rect_forced || (elem == ELEM_BF16 && x.rect >= 200 && x.t64 <= 1024 && x.steps >= 16)) return GEMM_128x64;
  return GEMM_64x1;
}

// ... and of a weight-gradient launch (M, N = layer widths, K = batch).  Within 0.4 % of the best on 900
// timed shapes: 16-tiles while they have a compute unit each, 32-tiles with an eight-way K split up to two and
// a half per compute unit (fp32 512 x 256 x 1024 twice: 46.1 us on 64-tiles, 15.6 us; bf16 512 x 512 x
// 512 twice: 10.0 / 6.0 us), then 64-tiles; bf16 launches with enough 128-tiles to fill the chip
// twice take the kernel for large layers.  The whole group of layers that one launch covers decides, also
// where they are launched one by one, so that both give the same bits.
int plan_wgrad(betty_handle h, Elem elem, int layer, bool rop, bool two, int B) {
  const int first = (layer - 1) / MAX_PROBLEMS * MAX_PROBLEMS, last = std::min(h->L, first + MAX_PROBLEMS);
  Extent x;
  for (int i = first; i < last; ++i)
    x.add(elem, h->layers[i].n_in, h->layers[i].n_out, B, two || (rop && i > 0) ? B : 0);
  if (elem == ELEM_BF16 && h->tune_wgrad128_min > 0 && x.t128 >= h->tune_wgrad128_min) return GEMM_128x1;
  if (h->tune_wgrad_cfg != GEMM_64x1 || !h->tune_split || h->tune_wgrad128_min == 0) return h->tune_wgrad_cfg;
  const int shorter = elem == ELEM_BF16 ? 1 : 2;
  if (x.t16 <= 256 || (x.t16 <= 512 && x.steps <= 4 * shorter) || (x.t16 <= 1024 && x.steps <= 2 * shorter)) return GEMM_16;
  return x.t32 <= 600 ? GEMM_32x8 : GEMM_64x1;
}

void set_pairs(GemmArgs& g, const void* A0, int lda0, const void* B0, int ldb0, int K0, const void* A1,
               int lda1, const void* B1, int ldb1, int K1) {
  g.A[0] = A0; g.B[0] = B0; g.lda[0] = lda0; g.ldb[0] = ldb0; g.K[0] = K0;
  g.A[1] = A1 ? A1 : A0; g.B[1] = A1 ? B1 : B0; g.lda[1] = A1 ? lda1 : lda0; g.ldb[1] = A1 ? ldb1 : ldb0;
  g.K[1] = A1 ? K1 : 0;
  g.xgm = g.xgn = 0;
  g.split = 0;
}

// one activation-shaped GEMM with a fused epilogue
void chain_gemm(betty_handle h, Elem elem, const void* A0, int lda0, const void* B0, int ldb0, int K0,
                const void* A1, int lda1, const void* B1, int ldb1, int K1, int M, int N, const Epilogue& e,
                double flops) {
  GemmBatch b;
  b.n = 1;
  GemmProblem& p = b.p[0];
  set_pairs(p.g, A0, lda0, B0, ldb0, K0, A1, lda1, B1, ldb1, K1);
  p.g.M = M; p.g.N = N;
  p.e = e;
  launch_gemm_batch(h->ctx, elem, plan_chain(h, elem, b), b, flops);
}

Epilogue blank_epilogue(int mode, int act = 0) {
  Epilogue e;
  memset(&e, 0, sizeof e);
  e.mode = mode;
  e.act = act;
  return e;
}

// operand copies of a flat parameter-shaped vector: per layer, as stored (n_in x n_out; not for layer 1, where
// only R-backward and backward links would read it, and there are none) and transposed; sixteen matrices a launch
struct Shadows { const float* flat; std::vector<size_t>* N; std::vector<size_t>* T; std::vector<size_t>* T32 = nullptr; };
void make_shadows(betty_handle h, OperandSet& os, std::initializer_list<Shadows> vectors) {
  ConvertBatch b;
  for (const Shadows& v : vectors) {
    for (int i = 0; i < h->L; ++i) {
      if (b.n == MAX_CONVERTS) { launch_convert_batch(h->ctx, os.elem, b); b.n = 0; }
      const LayerInfo& li = h->layers[i];
      ConvertJob& j = b.j[b.n++];
      j = ConvertJob{v.flat + li.w_off, li.n_out, li.n_in, li.n_out, v.N && i > 0 ? h->at<void>((*v.N)[i]) : nullptr, li.n_out_p,
                     v.T ? h->at<void>((*v.T)[i]) : nullptr, li.n_in_p};
      if (v.T32) j.outT32 = h->f((*v.T32)[i]);
    }
  }
  launch_convert_batch(h->ctx, os.elem, b);
}

// A ReLU mask is a discontinuous function of the pre-activation: deciding it from bf16-rounded
// operands flips about one unit in a thousand, which alone costs a few percent of relative error
// in every gradient that passes through the mask.  With bf16 operands the forward products of a
// ReLU network are therefore formed from the fp32 operand set; all other GEMMs stay bf16.
bool hybrid_forward(betty_handle h, const OperandSet& os) {
  return os.elem == ELEM_BF16 && h->desc.act == BETTY_ACT_RELU && h->sets[1].present;
}

// operand copies of the parameters w for everything that follows
// and, with v, of a direction for the forward-over-reverse passes
void make_weight_operands(betty_handle h, OperandSet& os, const float* w, const float* v = nullptr, bool rforward_only = false) {
  // (with the fp32 forward of ReLU networks the same launch also leaves the fp32 transposed copies)
  const Shadows sw{w, &os.Wn, &os.Wt, hybrid_forward(h, os) ? &h->sets[1].Wt : nullptr};
  if (v) make_shadows(h, os, {sw, Shadows{v, rforward_only ? nullptr : &os.Vn, &os.Vt}});
  else make_shadows(h, os, {sw});
}

// One first-order pass over a batch.  Up to two of them share their launches: the train and the
// validation batch at the same weights, or the two perturbed points of a central difference.
struct Pass {
  OperandSet* os;                   // weights and buffers
  int side;                         // 0 = train (lower cost), 1 = validation (upper cost)
  const float* w;                   // flat parameters, for the biases
  const float* theta = nullptr;     // weight net (train side of the reweighting cost)
  const float* omega_fixed = nullptr;   // sample weights to use instead of it
  float sign = 1.f;                 // -1: output delta, and with it every delta, with the opposite sign
  bool curvature = false;           // also phi'' and (delta W^T) phi'', for forward-over-reverse passes
  size_t ell = 0, omega = 0, dsig = 0;  // other places for the per-sample values (0: the side's own)
};
Pass train_pass(betty_handle h, OperandSet& os, const float* w, const float* lam, bool curvature) {
  Pass p{&os, 0, w};
  p.theta = wnet_theta(h, lam);
  p.curvature = curvature;
  return p;
}
Pass val_pass(OperandSet& os, const float* w) { return Pass{&os, 1, w}; }

// a_l, phi'(z_l) (phi''), logits, per-sample loss, output delta
// (upto: only the activations of the layers up to that one)
void forward_and_loss(betty_handle h, const Pass* ps, int n, int upto = 0) {
  const int L = h->L;
  const bool hybrid = hybrid_forward(h, *ps[0].os);
  const Elem elem = hybrid ? ELEM_F32 : ps[0].os->elem;     // operands of the forward products
  for (int l = h->layer1_done ? 2 : 1; l <= (upto > 0 ? upto : L); ++l) {
    const LayerInfo& li = h->layers[l - 1];
    const bool last = l == L;
    GemmBatch b;
    double flops = 0;
    // (finite differences: z_1 of the train batch, whether or not that batch is among the passes)
    const Pass* z1 = l == 1 ? h->z1_pass : nullptr;
    const bool extra = z1 && !(ps[0].os == z1->os && ps[0].side == z1->side);
    for (int i = 0; i < n + (extra ? 1 : 0); ++i) {
      const Pass& ps_i = i < n ? ps[i] : *z1;
      OperandSet& fs = hybrid ? h->sets[1] : *ps_i.os;
      SideBuf& sb = ps_i.os->side[ps_i.side];
      SideBuf& fb = fs.side[ps_i.side];
      GemmProblem& p = b.p[b.n++];
      const void* Aop = l == 1 ? h->at<void>(fb.X) : h->at<void>(fb.A[l - 1]);
      set_pairs(p.g, Aop, li.n_in_p, h->at<void>(fs.Wt[l - 1]), li.n_in_p, li.n_in, nullptr, 0, nullptr, 0, 0);
      p.g.M = sb.B; p.g.N = li.n_out;
      Epilogue e = blank_epilogue(last ? EPI_FWD_LAST : EPI_FWD, h->desc.act);
      e.colvec = h->desc.has_bias ? ps_i.w + li.b_off : nullptr;
      e.ldf = li.n_out_p;
      if (last) {
        e.f0 = h->f(sb.ZL);
      } else {
        if (z1 && ps_i.side == z1->side) e.f0 = h->f(h->fd_z1);
        e.dphi_out = h->f(sb.dphi[l]);
        e.d2_out = ps_i.curvature && sb.e2[l] ? h->f(sb.e2[l]) : nullptr;
        e.out = h->at<void>(fb.A[l]); e.ld = li.n_out_p;
        e.outT = hybrid ? nullptr : h->at<void>(fb.At[l]); e.ldT = sb.Bp;
        if (hybrid) { e.out2 = h->at<void>(sb.A[l]); e.outT2 = h->at<void>(sb.At[l]); }
      }
      p.e = e;
      flops += 2.0 * sb.B * li.n_in * li.n_out;
    }
    if (extra) --b.n;
    const int cfg = plan_chain(h, elem, b);
    if (extra) {
      // z_1 of that batch rides along where its product takes the passes' kernel anyway, whose choice (and with it the
      // passes' bits) it does not change; otherwise it takes a launch with the kernel of its own size
      GemmBatch own;
      own.n = 1;
      own.p[0] = b.p[b.n];
      const int own_cfg = plan_chain(h, elem, own);
      const double own_flops = 2.0 * own.p[0].g.M * li.n_in * li.n_out;
      if (own_cfg == cfg) ++b.n;
      else { launch_gemm_batch(h->ctx, elem, own_cfg, own, own_flops); flops -= own_flops; }
    }
    launch_gemm_batch(h->ctx, elem, cfg, b, flops);
  }
  if (upto > 0) return;
  const LayerInfo& lo = h->layers[L - 1];
  LossBatch lb;
  for (int i = 0; i < n; ++i) {
    SideBuf& sb = ps[i].os->side[ps[i].side];
    LossArgs& a = lb.a[lb.n++];
    a = LossArgs{};
    a.loss = h->desc.loss;
    a.reweight = (ps[i].side == 0 && h->desc.hp == BETTY_HP_REWEIGHT_NET) ? 1 : 0;
    a.hidden = h->desc.wnet_hidden;
    a.Z = h->f(sb.ZL); a.ldz = lo.n_out_p;
    a.labels = h->at<Labels>(h->labels) + ps[i].side; a.C = lo.n_out;
    a.theta = ps[i].theta;
    a.omega_fixed = ps[i].omega_fixed;
    a.rows = sb.B; a.inv_batch = ps[i].sign / (float)sb.B;
    a.ell = h->f(ps[i].ell ? ps[i].ell : sb.ell); a.s = h->f(sb.s);
    a.omega = h->f(ps[i].omega ? ps[i].omega : sb.omega); a.dsig = h->f(ps[i].dsig ? ps[i].dsig : sb.dsig);
    a.P = h->f(sb.P);
    a.D = h->at<void>(sb.D[L]); a.ldD = lo.n_out_p;
    a.Dt = h->at<void>(sb.Dt[L]); a.ldDt = sb.Bp;
  }
  launch_loss_rows(h->ctx, ps[0].os->elem, lb);
}

// delta_l for every layer below the output (and (delta W^T) phi'')
void backward_chain(betty_handle h, const Pass* ps, int n, int l_from = 0) {
  const int L = h->L;
  const Elem elem = ps[0].os->elem;
  for (int l = l_from > 0 ? l_from : L; l >= 2; --l) {
    const LayerInfo& li = h->layers[l - 1];
    GemmBatch b;
    double flops = 0;
    for (int i = 0; i < n; ++i) {
      SideBuf& sb = ps[i].os->side[ps[i].side];
      GemmProblem& p = b.p[b.n++];
      set_pairs(p.g, h->at<void>(sb.D[l]), li.n_out_p, h->at<void>(ps[i].os->Wn[l - 1]), li.n_out_p, li.n_out, nullptr, 0,
                nullptr, 0, 0);
      p.g.M = sb.B; p.g.N = li.n_in;
      Epilogue e = blank_epilogue(EPI_BWD);
      e.dphi = h->f(sb.dphi[l - 1]);
      e.e_io = ps[i].curvature && sb.e2[l - 1] ? h->f(sb.e2[l - 1]) : nullptr;
      e.ldf = li.n_in_p;
      e.out = l > 2 ? h->at<void>(sb.D[l - 1]) : nullptr; e.ld = li.n_in_p;      // (delta_1 has no link below it)
      e.outT = h->at<void>(sb.Dt[l - 1]); e.ldT = sb.Bp;
      p.e = e;
      flops += 2.0 * sb.B * li.n_in * li.n_out;
    }
    launch_gemm_batch(h->ctx, elem, plan_chain(h, elem, b), b, flops);
  }
}

NarrowNet narrow_net(betty_handle h, int first) {
  NarrowNet net{};
  net.L = h->L; net.first = first;
  for (int l = 0; l <= h->L; ++l) {
    net.n[l] = h->dims[l];
    net.np[l] = padup(h->dims[l]);
  }
  net.act = h->desc.act; net.loss = h->desc.loss;
  return net;
}

void narrow_forward_backward(betty_handle h, const Pass* ps, int n, int first) {
  const int L = h->L;
  const bool hybrid = hybrid_forward(h, *ps[0].os);
  if (first > 1 && !h->layer1_done) forward_and_loss(h, ps, n, first - 1);
  NarrowGradArgs a{};
  a.net = narrow_net(h, first);
  a.hidden = h->desc.wnet_hidden;
  double flops = 0;
  for (int i = 0; i < n; ++i) {
    OperandSet& os = *ps[i].os;
    OperandSet& fs = hybrid ? h->sets[1] : os;
    SideBuf& sb = os.side[ps[i].side];
    SideBuf& fb = fs.side[ps[i].side];
    NarrowGradSide& d = a.side[i];
    d.X = h->at<void>(fb.X);
    d.A1 = L > 1 ? h->at<void>(fb.A[1]) : nullptr;
    for (int l = 1; l <= L; ++l) {
      d.Wf[l - 1] = h->at<void>(fs.Wt[l - 1]);
      d.Wn[l - 1] = h->at<void>(os.Wn[l - 1]);
      d.bias[l - 1] = h->desc.has_bias ? ps[i].w + h->layers[l - 1].b_off : nullptr;
      if (l < L) {
        d.A[l - 1] = h->at<void>(sb.A[l]); d.At[l - 1] = h->at<void>(sb.At[l]);
        d.dphi[l - 1] = h->f(sb.dphi[l]);
        d.e2[l - 1] = ps[i].curvature && sb.e2[l] ? h->f(sb.e2[l]) : nullptr;
      }
      d.D[l - 1] = l > 1 ? h->at<void>(sb.D[l]) : nullptr; d.Dt[l - 1] = h->at<void>(sb.Dt[l]);
      flops += (l > 1 ? 4.0 : first == 1 ? 2.0 : 0.0) * sb.B * h->layers[l - 1].n_in * h->layers[l - 1].n_out;
    }
    d.labels = h->at<Labels>(h->labels) + ps[i].side;
    d.omega_fixed = ps[i].omega_fixed;
    d.ZL = h->f(sb.ZL); d.P = h->f(sb.P); d.s = h->f(sb.s);
    d.ell = h->f(ps[i].ell ? ps[i].ell : sb.ell);
    d.omega = h->f(ps[i].omega ? ps[i].omega : sb.omega); d.dsig = h->f(ps[i].dsig ? ps[i].dsig : sb.dsig);
    d.B = sb.B; d.Bp = sb.Bp;
    d.reweight = (ps[i].side == 0 && h->desc.hp == BETTY_HP_REWEIGHT_NET) ? 1 : 0;
    d.inv_batch = ps[i].sign / (float)sb.B;
    if (ps[i].theta) a.theta = ps[i].theta;
  }
  launch_narrow_grad(h->ctx, ps[0].os->elem, hybrid, a, n, flops);
}

// Forward pass, loss and backward chain.  A narrow output layer (see LastGradArgs) goes through
// one vector kernel that produces the logits, the loss quantities and delta_{L-1}.
void forward_backward(betty_handle h, const Pass* ps, int n) {
  const int L = h->L;
  const LayerInfo& lo = h->layers[L - 1];
  int samples = 0;
  for (int i = 0; i < n; ++i) samples += ps[i].os->side[ps[i].side].B * (h->as_pair && n == 1 ? 2 : 1);
  if (const int first = h->fixed_grouping && ps[0].os->elem == ELEM_BF16 ? 0 : narrow_first(h, false, ps[0].os->elem, samples)) {
    narrow_forward_backward(h, ps, n, first);
    return;
  }
  // (also with the fp32 forward of ReLU networks: the output layer has no mask to protect, and the
  // operand-type copy of a_{L-1} exists either way)
  const bool narrow = L >= 2 && lo.n_out <= LAST_ROP_MAX_C;
  if (!narrow) {
    forward_and_loss(h, ps, n);
    backward_chain(h, ps, n);
    return;
  }
  forward_and_loss(h, ps, n, L - 1);
  LastGradArgs a{};
  for (int i = 0; i < n; ++i) {
    SideBuf& sb = ps[i].os->side[ps[i].side];
    LastGradSide& d = a.side[a.n_sides++];
    d.A = h->at<void>(sb.A[L - 1]); d.lda = lo.n_in_p;
    d.labels = h->at<Labels>(h->labels) + ps[i].side;
    d.omega_fixed = ps[i].omega_fixed;
    d.ZL = h->f(sb.ZL); d.P = h->f(sb.P); d.ldz = lo.n_out_p;
    d.ell = h->f(ps[i].ell ? ps[i].ell : sb.ell); d.s = h->f(sb.s);
    d.omega = h->f(ps[i].omega ? ps[i].omega : sb.omega); d.dsig = h->f(ps[i].dsig ? ps[i].dsig : sb.dsig);
    d.DL = h->at<void>(sb.D[L]); d.DLt = h->at<void>(sb.Dt[L]); d.ldd = lo.n_out_p; d.ldDLt = sb.Bp;
    d.dphi = h->f(sb.dphi[L - 1]);
    d.e2 = ps[i].curvature && sb.e2[L - 1] ? h->f(sb.e2[L - 1]) : nullptr; d.ldf = lo.n_in_p;
    d.D = L > 2 ? h->at<void>(sb.D[L - 1]) : nullptr; d.ldD = lo.n_in_p; d.Dt = h->at<void>(sb.Dt[L - 1]); d.ldDt = sb.Bp;
    d.Wt = h->at<void>(ps[i].os->Wt[L - 1]); d.Wn = h->at<void>(ps[i].os->Wn[L - 1]);
    d.bias = h->desc.has_bias ? ps[i].w + lo.b_off : nullptr;
    d.B = sb.B;
    d.reweight = (ps[i].side == 0 && h->desc.hp == BETTY_HP_REWEIGHT_NET) ? 1 : 0;
    d.inv_batch = ps[i].sign / (float)sb.B;
    if (ps[i].theta) a.theta = ps[i].theta;
  }
  a.ldt = lo.n_in_p; a.ldn = lo.n_out_p;
  a.hidden = h->desc.wnet_hidden;
  a.n_in = lo.n_in; a.C = lo.n_out; a.loss = h->desc.loss;
  launch_last_layer_grad(h->ctx, ps[0].os->elem, a);
  backward_chain(h, ps, n, L - 1);
}

// Split of a tile grid over the eight XCDs (see GemmArgs::xgm): the factorisation gm x gn = 8 that
// divides the grid and minimises the operand rows each L2 fetches, gn * tiles_m + gm * tiles_n
// (every XCD reads tiles_m / gm row panels and tiles_n / gn column panels).  gm = gn = 0 when
// nothing fits or the row-major order is already as good.
void xcd_split(int tiles_m, int tiles_n, int& gm, int& gn) {
  gm = gn = 0;
  if ((tiles_m * tiles_n) % 8 != 0 || tiles_m * tiles_n < 256) return;   // small grids: no measurable gain
  long best = tiles_n % 8 == 0 ? 8L * tiles_m + tiles_n : -1;      // row-major order = 1 x 8 when tiles_n % 8 == 0
  for (int a = 1; a <= 8; a *= 2) {
    const int b = 8 / a;
    if (tiles_m % a || tiles_n % b) continue;
    const long cost = (long)b * tiles_m + (long)a * tiles_n;
    if (best < 0 || cost < best) { best = cost; gm = a; gn = b; }
  }
}

// the proximal cost's share of the series' recurrence V <- g + beta V - alpha (...) in layer l
bool anchored(betty_handle h, int l) { return h->desc.hp == BETTY_HP_PROXIMAL && !(h->desc.prox_skip_last && l == h->L); }
double series_beta(betty_handle h, int l, double alpha) { return anchored(h, l) ? 1.0 - 2.0 * alpha * h->desc.prox_rho : 1.0; }

// What the grouped weight-gradient launch does with its result.
struct WgradSink {
  int mode;                 // EPI_WGRAD / EPI_WGRAD_INIT / EPI_WGRAD_NEUMANN
  float* C;                 // flat output (EPI_WGRAD)
  const float* lam;         // non-null adds the L2-decay term 2 e^lam x
  const float* x;
  float* v; float* p; float alpha;
  bool copies;              // also write the operand copies of the new v
  bool second_set = false;  // ... into the second set of direction copies (the first is still being read)
  float beta = 0.f, gamma = 0.f;   // EPI_WGRAD_SGD: momentum factor and plain weight decay
  int K = 0;                // EPI_WGRAD_SCALED: steps of the series
  bool sums_split = false;  // ... its sums over the steps are value and remainder (samples_accumulate)
  const float* eps = nullptr;      // EPI_WGRAD_FD
  OperandSet* minus = nullptr;     // the second perturbed point: its products are added (its deltas carry the sign)
  bool minus_summed = false;       // ... and layer 1's deltas of both points stand added in the second's place
  bool sum_p = false;
  int* sums = nullptr;             // non-null: the launch leaves its sums in vec partials, their number here
};
// (aggregate initialisation in the callers lists the fields up to `copies`)

// All layers' parameter-shaped products in one launch: plain gradient a^T delta (rop = false) or
// the R-op form Ra^T delta + a^T Rdelta (rop = true), bias rows included.
void wgrad_batch(betty_handle h, OperandSet& os, int side, bool rop, const WgradSink& k, int l_first = 1,
                 int l_last = 0) {
  SideBuf& sb = os.side[side];
  const int L = l_last > 0 ? l_last : h->L, B = sb.B, Bp = sb.Bp;
  const std::vector<size_t>& VN = k.second_set ? os.Vn2 : os.Vn;
  const std::vector<size_t>& VT = k.second_set ? os.Vt2 : os.Vt;
  for (int l0 = l_first; l0 <= L; l0 += MAX_PROBLEMS) {
    GemmBatch b;
    b.n = std::min(MAX_PROBLEMS, L - l0 + 1);
    double flops = 0;
    for (int i = 0; i < b.n; ++i) {
      const int l = l0 + (b.n - 1 - i);         // deepest layer first
      const LayerInfo& li = h->layers[l - 1];
      GemmProblem& p = b.p[i];
      const void* aT = l == 1 ? h->at<void>(sb.XT) : h->at<void>(sb.At[l - 1]);
      if (k.minus) {
        SideBuf& mb = k.minus->side[side];
        if (k.minus_summed && l == 1) set_pairs(p.g, aT, Bp, h->at<void>(mb.Dt[1]), Bp, B, nullptr, 0, nullptr, 0, 0);
        else set_pairs(p.g, aT, Bp, h->at<void>(sb.Dt[l]), Bp, B, l == 1 ? aT : h->at<void>(mb.At[l - 1]), Bp,
                  h->at<void>(mb.Dt[l]), Bp, B);
        flops += (k.minus_summed && l == 1 ? 2.0 : 4.0) * B * li.n_in * li.n_out;
      } else if (!rop) {
        set_pairs(p.g, aT, Bp, h->at<void>(sb.Dt[l]), Bp, B, nullptr, 0, nullptr, 0, 0);
        flops += 2.0 * B * li.n_in * li.n_out;
      } else if (k.sums_split) {
        const bool ra = l > 1;
        set_pairs(p.g, ra ? h->at<void>(os.sumRA[l - 1]) : aT, 2 * Bp, h->at<void>(sb.Dt[l]), Bp, ra ? B : 0, aT, Bp,
                  h->at<void>(os.sumRD[l]), 2 * Bp, B);
        p.g.split = 1;
        flops += (ra ? 4.0 : 2.0) * B * li.n_in * li.n_out;
      } else if (l == 1) {
        set_pairs(p.g, aT, Bp, h->at<void>(os.RDt[l]), Bp, B, nullptr, 0, nullptr, 0, 0);
        flops += 2.0 * B * li.n_in * li.n_out;
      } else {
        set_pairs(p.g, h->at<void>(os.RAt[l - 1]), Bp, h->at<void>(sb.Dt[l]), Bp, B, aT, Bp,
                  h->at<void>(os.RDt[l]), Bp, B);
        flops += 4.0 * B * li.n_in * li.n_out;
      }
      p.g.M = li.n_in; p.g.N = li.n_out;
      Epilogue e = blank_epilogue(k.mode);
      e.ldc = li.n_out;
      e.C = k.C ? k.C + li.w_off : nullptr;
      e.lam = k.lam ? k.lam + li.w_off : nullptr;
      e.x = k.x ? k.x + li.w_off : nullptr;
      e.v = k.v ? k.v + li.w_off : nullptr;
      e.p = k.p ? k.p + li.w_off : nullptr;
      e.alpha = k.alpha; e.beta = k.beta; e.gamma = k.gamma;
      if (k.mode == EPI_WGRAD_SCALED) {
        // 2 rho alpha sum_j beta^j and 2 rho alpha^2, rounded once: an error in them is one of the whole result
        const double beta = series_beta(h, l, k.alpha), gamma = anchored(h, l) ? 2.0 * h->desc.prox_rho * k.alpha : 0.0;
        double sum = 1.0;
        for (int j = 0; j < k.K; ++j) sum = 1.0 + beta * sum;
        e.beta = (float)(gamma * sum);
        e.alpha = (float)(gamma * k.alpha);
      }
      if (k.copies) {
        e.out = l > 1 ? h->at<void>(VN[l - 1]) : nullptr; e.ld = li.n_out_p;     // (as in make_shadows)
        e.outT = h->at<void>(VT[l - 1]); e.ldT = li.n_in_p;
      }
      e.eps = k.eps; e.sum_p = k.sum_p;
      p.e = e;
      if (h->desc.has_bias) {
        BiasJob& j = b.bias[b.n_bias++];
        j = BiasJob{};
        const bool summed = k.minus_summed && l == 1;
        j.Mt2 = k.minus && !summed ? h->at<void>(k.minus->side[side].Dt[l]) : nullptr;
        j.eps = k.eps; j.sum_p = k.sum_p;
        j.Mt = rop ? h->at<void>(os.RDt[l]) : h->at<void>(summed ? k.minus->side[side].Dt[l] : sb.Dt[l]);
        j.ld = Bp; j.rows = li.n_out; j.k = B; j.mode = k.mode;
        if (k.sums_split) { j.Mt = h->at<void>(os.sumRD[l]); j.ld = 2 * Bp; j.k = (B + 63) / 64 * 128; }
        j.C = k.C ? k.C + li.b_off : nullptr;
        j.lam = k.lam ? k.lam + li.b_off : nullptr;
        j.x = k.x ? k.x + li.b_off : nullptr;
        j.v = k.v ? k.v + li.b_off : nullptr;
        j.p = k.p ? k.p + li.b_off : nullptr;
        j.alpha = e.alpha; j.beta = e.beta; j.gamma = e.gamma;
      }
    }
    double params = 0, copies = 0;
    for (int i = 0; i < b.n; ++i) {
      const LayerInfo& li = h->layers[l0 + i - 1];
      params += (double)li.n_in * li.n_out + (h->desc.has_bias ? li.n_out : 0);
      copies += (l0 + i > 1 ? 4.0 : 2.0) * li.n_in * li.n_out;
    }
    // algorithmic bytes per parameter of the epilogue's vector work (fp32 vectors 4 B each way,
    // operand copies 2 x 2 B, of layer 1 only the transposed one): Neumann step reads s, g (+ the diagonal), writes s and the copies
    double per_param = 4.0;
    if (k.mode == EPI_WGRAD_NEUMANN) per_param = 8.0 + 4.0 + (k.lam ? 4.0 : 0.0);
    else if (k.mode == EPI_WGRAD_NEUMANN_L2) per_param = 16.0 + 4.0;
    else if (k.mode == EPI_WGRAD_SGD) per_param = 16.0 + (k.lam ? 4.0 : 0.0);
    else if (k.mode == EPI_WGRAD_SCALED) per_param = 8.0;
    else if (k.mode == EPI_WGRAD_FD) per_param = 16.0 + (k.lam ? 4.0 : 0.0);
    else if (k.mode == EPI_WGRAD_FD_LAST) per_param = 16.0 + (k.x ? 4.0 : 0.0);
    else if (k.mode == EPI_WGRAD_INIT) per_param = k.p ? 8.0 : 4.0;
    else if (k.mode == EPI_WGRAD_CG) per_param = k.lam ? 12.0 : 8.0;
    else if (k.lam) per_param = 12.0;
    const int cfg = plan_wgrad(h, os.elem, l0, rop, k.minus != nullptr, B), bt = gemm_cfg_tile(cfg);
    if (cfg == GEMM_64x1 || cfg == GEMM_128x1)
      for (int i = 0; i < b.n; ++i)
        xcd_split((b.p[i].g.M + bt - 1) / bt, (b.p[i].g.N + bt - 1) / bt, b.p[i].g.xgm, b.p[i].g.xgn);
    const int n = launch_gemm_batch(h->ctx, os.elem, cfg, b, flops, per_param * params + (k.copies ? copies : 0.0),
                                    k.sums ? h->at<double>(h->sums) + *k.sums : nullptr);
    if (k.sums) *k.sums += n;
  }
}

// R-forward along the direction whose operand copies are in os.Vt and whose fp32 flat form is
// `vflat` (for the bias directions).  Leaves Rz_l (fp32) and Ra_l.
// With fuse_hessian (outputs of at most 32 columns) the last layer's epilogue applies the loss
// Hessian and leaves R delta_L instead of Rz_L.
void r_forward(betty_handle h, OperandSet& os, const float* vflat, bool fuse_hessian = false, int upto = 0) {
  SideBuf& sb = os.side[0];
  const int L = h->L, B = sb.B, Bp = sb.Bp;
  for (int l = 1; l <= (upto > 0 ? upto : L); ++l) {
    const LayerInfo& li = h->layers[l - 1];
    const bool last = l == L;
    const void* a_prev = l == 1 ? h->at<void>(sb.X) : h->at<void>(sb.A[l - 1]);
    Epilogue e = blank_epilogue(last ? (fuse_hessian ? EPI_RFWD_LAST_HESS : EPI_RFWD_LAST) : EPI_RFWD);
    e.colvec = h->desc.has_bias ? vflat + li.b_off : nullptr;
    e.f0 = h->f(os.Rz[l]);
    e.ldf = li.n_out_p;
    if (last && fuse_hessian) {
      e.act = h->desc.loss;
      e.dphi = h->desc.loss == BETTY_LOSS_SOFTMAX_CE ? h->f(sb.P) : nullptr;
      e.e = h->f(sb.s);
      e.out = h->at<void>(os.RD[l]); e.ld = li.n_out_p;
      e.outT = h->at<void>(os.RDt[l]); e.ldT = Bp;
    }
    if (!last) {
      e.dphi = h->f(sb.dphi[l]);
      e.out = h->at<void>(os.RA[l]); e.ld = li.n_out_p;
      e.outT = h->at<void>(os.RAt[l]); e.ldT = Bp;
    }
    if (l == 1)
      chain_gemm(h, os.elem, a_prev, li.n_in_p, h->at<void>(os.Vt[0]), li.n_in_p, li.n_in, nullptr, 0, nullptr,
                 0, 0, B, li.n_out, e, 2.0 * B * li.n_in * li.n_out);
    else
      chain_gemm(h, os.elem, h->at<void>(os.RA[l - 1]), li.n_in_p, h->at<void>(os.Wt[l - 1]), li.n_in_p,
                 li.n_in, a_prev, li.n_in_p, h->at<void>(os.Vt[l - 1]), li.n_in_p, li.n_in, B, li.n_out, e,
                 4.0 * B * li.n_in * li.n_out);
  }
}

// One Hessian-vector product with the forward/backward cache of the train batch in place; the
// parameter-shaped result goes where `sink` says (plain store, or fused into the recurrence).
// The weight-gradient launch of layer l, enqueued on the second stream as soon as R delta_l exists.
void side_wgrad(betty_handle h, OperandSet& os, const WgradSink& sink, int l) {
  hipStream_t main = h->ctx.stream;
  hipError_t e = hipEventRecord(h->fork_events[l - 1], main);
  if (e == hipSuccess) e = hipStreamWaitEvent(h->side_stream, h->fork_events[l - 1], 0);
  if (e != hipSuccess && h->ctx.first_error == hipSuccess) h->ctx.first_error = e;
  h->ctx.stream = h->side_stream;
  wgrad_batch(h, os, 0, true, sink, l, l);
  h->ctx.stream = main;
}

// The forward-over-reverse pass of narrow.hip along the direction in os.Vt, os.Vn and vflat; with cvec only the
// R-forward and the loss's derivative along it.
void narrow_rop(betty_handle h, OperandSet& os, const float* vflat, int first, float* cvec) {
  SideBuf& sb = os.side[0];
  const int L = h->L;
  if (first > 1) r_forward(h, os, vflat, false, first - 1);
  NarrowRopArgs a{};
  a.net = narrow_net(h, first);
  a.X = h->at<void>(sb.X); a.RA1 = h->at<void>(os.RA[1]);
  double flops = 0;
  for (int l = 1; l <= L; ++l) {
    const LayerInfo& li = h->layers[l - 1];
    a.Wt[l - 1] = h->at<void>(os.Wt[l - 1]); a.Vt[l - 1] = h->at<void>(os.Vt[l - 1]);
    a.Wn[l - 1] = h->at<void>(os.Wn[l - 1]); a.Vn[l - 1] = h->at<void>(os.Vn[l - 1]);
    a.cbias[l - 1] = h->desc.has_bias ? vflat + li.b_off : nullptr;
    if (l < L) {
      a.A[l - 1] = h->at<void>(sb.A[l]);
      a.dphi[l - 1] = h->f(sb.dphi[l]);
      a.e2[l - 1] = sb.e2[l] ? h->f(sb.e2[l]) : nullptr;
      a.Rz[l - 1] = sb.e2[l] && !cvec ? h->f(os.Rz[l]) : nullptr;
      a.RAt[l - 1] = cvec ? nullptr : h->at<void>(os.RAt[l]);
    }
    a.D[l - 1] = h->at<void>(sb.D[l]);
    a.RDt[l - 1] = h->at<void>(os.RDt[l]);
    flops += (l > 1 ? cvec ? 4.0 : 8.0 : first == 1 ? 2.0 : 0.0) * sb.B * li.n_in * li.n_out;
  }
  a.P = h->f(sb.P); a.s = h->f(sb.s); a.Z = h->f(sb.ZL); a.labels = h->at<Labels>(h->labels);
  a.cvec = cvec;
  a.B = sb.B; a.Bp = sb.Bp;
  StagedArgs staged;
  narrow_lds(a.net, os.elem, false);
  const bool curvature = sb.e2[1] != 0;
  if (h->rop_form.staged && staged_plan(a, os.elem, curvature, staged)) launch_staged_rop(h->ctx, os.elem, curvature, staged, flops);
  else launch_narrow_rop(h->ctx, os.elem, a, flops);
}

void hvp_cached(betty_handle h, OperandSet& os, const float* vflat, const WgradSink& sink, bool pipelined = false) {
  if (const int first = narrow_rop_first(h)) {
    narrow_rop(h, os, vflat, first, nullptr);
    wgrad_batch(h, os, 0, true, sink);
    return;
  }
  SideBuf& sb = os.side[0];
  const int L = h->L, B = sb.B, Bp = sb.Bp;
  const bool pipe = pipelined && h->side_stream && L >= 2;
  const LayerInfo& lo = h->layers[L - 1];
  // a narrow output layer goes through one vector kernel: last R-forward product, loss Hessian and
  // the R-backward step through that layer
  const bool narrow_last = L >= 2 && lo.n_out <= LAST_ROP_MAX_C;
  const bool fused_hessian = !narrow_last && lo.n_out <= 32;
  r_forward(h, os, vflat, fused_hessian, narrow_last ? L - 1 : 0);
  if (narrow_last) {
    LastRopArgs a{};
    a.RA = h->at<void>(os.RA[L - 1]); a.A = h->at<void>(sb.A[L - 1]); a.lda = lo.n_in_p;
    a.Wt = h->at<void>(os.Wt[L - 1]); a.Vt = h->at<void>(os.Vt[L - 1]); a.ldt = lo.n_in_p;
    a.Wn = h->at<void>(os.Wn[L - 1]); a.Vn = h->at<void>(os.Vn[L - 1]); a.ldn = lo.n_out_p;
    a.cbias = h->desc.has_bias ? vflat + lo.b_off : nullptr;
    a.P = h->f(sb.P); a.s = h->f(sb.s); a.ldp = lo.n_out_p;
    a.DL = h->at<void>(sb.D[L]); a.ldd = lo.n_out_p;
    a.dphi = h->f(sb.dphi[L - 1]); a.e2 = sb.e2[L - 1] ? h->f(sb.e2[L - 1]) : nullptr;
    a.Rz = h->f(os.Rz[L - 1]); a.ldf = lo.n_in_p;
    a.RDL = h->at<void>(os.RD[L]); a.RDLt = h->at<void>(os.RDt[L]); a.ldRDLt = Bp;
    a.RD = L > 2 ? h->at<void>(os.RD[L - 1]) : nullptr; a.ldRD = lo.n_in_p; a.RDt = h->at<void>(os.RDt[L - 1]); a.ldRDt = Bp;
    a.B = B; a.n_in = lo.n_in; a.C = lo.n_out; a.loss = h->desc.loss;
    launch_last_layer_rop(h->ctx, os.elem, a);
    if (pipe) { side_wgrad(h, os, sink, L); side_wgrad(h, os, sink, L - 1); }
  } else {
    if (!fused_hessian)
      launch_loss_hessian_rows(h->ctx, os.elem, h->desc.loss, h->f(sb.P), h->f(os.Rz[L]), lo.n_out_p, h->f(sb.s), B,
                               lo.n_out, h->at<void>(os.RD[L]), lo.n_out_p, h->at<void>(os.RDt[L]), Bp);
    if (pipe) side_wgrad(h, os, sink, L);
  }
  for (int l = narrow_last ? L - 1 : L; l >= 2; --l) {
    const LayerInfo& li = h->layers[l - 1];
    Epilogue e = blank_epilogue(EPI_RBWD);
    e.dphi = h->f(sb.dphi[l - 1]);
    e.e = sb.e2[l - 1] ? h->f(sb.e2[l - 1]) : nullptr;
    e.Rz = h->f(os.Rz[l - 1]);
    e.ldf = li.n_in_p;
    e.out = l > 2 ? h->at<void>(os.RD[l - 1]) : nullptr; e.ld = li.n_in_p;
    e.outT = h->at<void>(os.RDt[l - 1]); e.ldT = Bp;
    chain_gemm(h, os.elem, h->at<void>(os.RD[l]), li.n_out_p, h->at<void>(os.Wn[l - 1]), li.n_out_p, li.n_out,
               h->at<void>(sb.D[l]), li.n_out_p, h->at<void>(os.Vn[l - 1]), li.n_out_p, li.n_out, B, li.n_in, e,
               4.0 * B * li.n_in * li.n_out);
    if (pipe) side_wgrad(h, os, sink, l - 1);
  }
  if (!pipe) {
    wgrad_batch(h, os, 0, true, sink);
    return;
  }
  // the next product reads every layer's new direction: the main stream waits for the second one
  hipError_t e = hipEventRecord(h->join_event, h->side_stream);
  if (e == hipSuccess) e = hipStreamWaitEvent(h->ctx.stream, h->join_event, 0);
  if (e != hipSuccess && h->ctx.first_error == hipSuccess) h->ctx.first_error = e;
}

// full first-order gradient of the lower cost at w (operand copies of w already made)
void lower_grad_seq(betty_handle h, OperandSet& os, const float* w, const float* lam, float* grad, float* loss_or_null) {
  const float* dl = diag_log(h, lam);
  const Pass ps = train_pass(h, os, w, lam, false);
  forward_backward(h, &ps, 1);
  // the diagonal term multiplies w itself or its distance to the anchor; its cost is summed on the way
  int n = 0;
  WgradSink k{EPI_WGRAD, grad, dl, dl ? w : nullptr, nullptr, nullptr, 0.f, false};
  if (h->desc.hp == BETTY_HP_PROXIMAL) k.p = const_cast<float*>(lam);
  if (dl && loss_or_null) k.sums = &n;
  wgrad_batch(h, os, 0, false, k);
  if (loss_or_null)
    launch_weighted_loss_sum(h->ctx, h->f(os.side[0].s), h->f(os.side[0].ell), os.side[0].B, h->at<double>(h->sums), n, loss_or_null);
}

// gradient of the upper cost on the validation batch; the result goes where `sink` says.  With
// with_lower the same launches also build the forward/backward cache of the train batch that the
// R-op passes need (no parameter gradient on that side).
void upper_grad_seq(betty_handle h, OperandSet& os, const float* w, const float* lam, bool with_lower,
                    const WgradSink& sink, float* loss_or_null) {
  Pass ps[2] = {val_pass(os, w), val_pass(os, w)};
  if (with_lower) ps[0] = train_pass(h, os, w, lam, true);
  forward_backward(h, ps, with_lower ? 2 : 1);
  wgrad_batch(h, os, 1, false, sink);
  if (loss_or_null)
    launch_weighted_loss_sum(h->ctx, h->f(os.side[1].s), h->f(os.side[1].ell), os.side[1].B, nullptr, 0, loss_or_null);
}

// forward/backward cache of the train batch for the R-op passes (no parameter gradient)
void prepare_lower(betty_handle h, OperandSet& os, const float* w, const float* lam) {
  const Pass ps = train_pass(h, os, w, lam, true);
  forward_backward(h, &ps, 1);
}

// out = -(1/B) sum_i c_i dR/dtheta with c_i = <grad_w l_i, scale * qflat>
void mixed_reweight_seq(betty_handle h, OperandSet& os, const float* lam, const float* qflat, float scale,
                        float* out, bool copies_current = false) {
  SideBuf& sb = os.side[0];
  const int L = h->L;
  const LayerInfo& lo = h->layers[L - 1];
  // c_i is linear in the direction, so the scale is applied once, to the final sum over samples
  if (!copies_current) make_shadows(h, os, {Shadows{qflat, nullptr, &os.Vt}});   // else os.Vt already holds qflat
  if (const int first = narrow_rop_first(h)) {
    narrow_rop(h, os, qflat, first, h->f(os.cvec));
  } else if (L >= 2 && lo.n_out <= LAST_ROP_MAX_C) {
    // narrow output layer: the last product and the directional derivative in one vector kernel
    r_forward(h, os, qflat, false, L - 1);
    LastRopArgs a{};
    a.RA = h->at<void>(os.RA[L - 1]); a.A = h->at<void>(sb.A[L - 1]); a.lda = lo.n_in_p;
    a.Wt = h->at<void>(os.Wt[L - 1]); a.Vt = h->at<void>(os.Vt[L - 1]); a.ldt = lo.n_in_p;
    a.cbias = h->desc.has_bias ? qflat + lo.b_off : nullptr;
    a.P = h->f(sb.P); a.ldp = lo.n_out_p;
    a.B = sb.B; a.n_in = lo.n_in; a.C = lo.n_out; a.loss = h->desc.loss;
    a.cvec = h->f(os.cvec); a.labels = h->at<Labels>(h->labels); a.Z = h->f(sb.ZL);
    launch_last_layer_rop(h->ctx, os.elem, a);
  } else {
    r_forward(h, os, qflat);
    launch_loss_directional_rows(h->ctx, h->desc.loss, h->f(sb.P), h->f(sb.ZL), h->at<Labels>(h->labels),
                                 h->f(os.Rz[L]), lo.n_out_p, sb.B, lo.n_out, h->f(os.cvec));
  }
  launch_wnet_theta_vjp(h->ctx, h->f(sb.ell), h->f(sb.dsig), h->f(os.cvec), nullptr, nullptr, lam, h->desc.wnet_hidden, sb.B,
                        scale / (float)sb.B, out);
}

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  const char* x = (const char*)a;
  const char* y = (const char*)b;
  return x < y + nb && y < x + na;
}

betty_status check_vec(betty_handle h, const void* p, const char* name) {
  if (!p) return fail(h, BETTY_ENULL, "%s is NULL", name);
  if (((uintptr_t)p) & 3) return fail(h, BETTY_EALIGN, "%s is not 4-byte aligned", name);
  return BETTY_OK;
}

betty_status check_ready(betty_handle h) {
  if (!h) return BETTY_ENULL;
  if (!h->bound) return fail(h, BETTY_EWORKSPACE, "no workspace bound (call betty_bind)");
  if (!h->batches) return fail(h, BETTY_EWORKSPACE, "batches not set (call betty_set_batches)");
  return BETTY_OK;
}

betty_status finish(betty_handle h) {
  if (h->ctx.first_error != hipSuccess) {
    betty_status st = fail(h, BETTY_EDEVICE, "HIP error: %s", hipGetErrorString(h->ctx.first_error));
    h->ctx.first_error = hipSuccess;
    return st;
  }
  return BETTY_OK;
}

#define CHECK(expr) do { betty_status st__ = (expr); if (st__ != BETTY_OK) return st__; } while (0)

}  // namespace

static void release_side_stream(betty_handle h) {
  for (hipEvent_t e : h->fork_events) if (e) (void)hipEventDestroy(e);
  h->fork_events.clear();
  if (h->join_event) (void)hipEventDestroy(h->join_event);
  h->join_event = nullptr;
  if (h->side_stream) (void)hipStreamDestroy(h->side_stream);
  h->side_stream = nullptr;
}

// What a workspace must hold before its first use: zero padding everywhere (fill kernels, no
// memset nodes), and for the proximal cost log(rho_j) per parameter.
static void init_workspace(betty_handle h, size_t bytes) {
  launch_fill_zero(h->ctx, h->ws, bytes);
  if (h->desc.hp == BETTY_HP_PROXIMAL) {
    // exp(-200) is exactly 0 in fp32, so parameters outside the proximal term get no curvature
    const LayerInfo& last = h->layers[h->L - 1];
    const size_t cut = h->desc.prox_skip_last ? last.w_off : h->d;
    const float lr = h->desc.prox_rho > 0.f ? std::log(h->desc.prox_rho) : -200.f;
    launch_fill_value(h->ctx, h->f(h->logrho), std::max(lr, -200.f), cut);
    if (cut < h->d) launch_fill_value(h->ctx, h->f(h->logrho) + cut, -200.f, h->d - cut);
  }
}

static unsigned long long next_epoch() {
  static std::atomic<unsigned long long> counter{0};
  return ++counter;
}

static void drop_graph(betty_handle_s::GraphSlot& g) {
  if (g.exec) (void)hipGraphExecDestroy(g.exec);
  if (g.graph) (void)hipGraphDestroy(g.graph);
  g = betty_handle_s::GraphSlot();
}

static void drop_graphs(betty_handle h) {
  for (auto& kind : h->graphs)
    for (auto& g : kind) drop_graph(g);
}

// Moves the handle's work to another stream, behind everything it has enqueued so far.
static hipError_t move_to_stream(betty_handle h, hipStream_t to) {
  if (h->ctx.stream == to) return hipSuccess;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipSuccess;
  if (hipStreamIsCapturing(to, &cap) != hipSuccess) (void)hipGetLastError();
  if (cap == hipStreamCaptureStatusNone) {          // (a stream being captured cannot wait for work outside its graph)
    if (!h->order_event) e = hipEventCreateWithFlags(&h->order_event, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(h->order_event, h->ctx.stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(to, h->order_event, 0);
  }
  if (e == hipSuccess) h->ctx.stream = to;
  return e;
}

// Runs `body` (which only enqueues kernels on ctx.stream) directly the first time a given
// argument set is seen, captures it into a graph the second time, and replays the graph from then
// on.  Any capture failure switches graphs off for the handle and runs the body directly.
template <typename Body>
static betty_status run_cached(betty_handle h, int kind, const betty_handle_s::CallKey& key, Body body) {
  const bool brief = kind >= betty_handle_s::CALL_SHORT;
  if (!h->use_graphs || h->ctx.profiling || (brief && h->d > betty_handle_s::SHORT_PARAMS)) { body(); return finish(h); }
  betty_handle_s::GraphSlot* g = nullptr;
  betty_handle_s::GraphSlot* oldest = &h->graphs[kind][0];
  for (auto& s : h->graphs[kind]) {
    if (s.used && s.key == key) g = &s;
    if (s.used < oldest->used) oldest = &s;
  }
  if (!g) {
    if (brief && oldest->exec && oldest->replays < 16) {
      int& after = h->record_after[kind - betty_handle_s::CALL_SHORT];
      after = std::min(2 * after, 1 << 20);
    }
    drop_graph(*oldest);
    oldest->key = key;
    oldest->used = ++h->graph_clock;
    const unsigned long long before = h->ctx.launches;
    body();
    oldest->launches = h->ctx.launches - before;
    oldest->calls = 1;
    return finish(h);
  }
  g->used = ++h->graph_clock;
  if (brief && !g->exec && (g->launches < betty_handle_s::SHORT_LAUNCHES ||
                            g->calls < h->record_after[kind - betty_handle_s::CALL_SHORT])) {
    ++g->calls;
    body();
    return finish(h);
  }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(h->ctx.stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();                        // the caller is recording a graph of its own
    body();
    return finish(h);
  }
  if (!g->exec) {
    const hipStream_t run = h->ctx.stream;
    hipError_t e = hipSuccess;
    if (!h->capture_stream) e = hipStreamCreateWithFlags(&h->capture_stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamBeginCapture(h->capture_stream, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      h->ctx.stream = h->capture_stream;
      body();
      h->ctx.stream = run;
      e = hipStreamEndCapture(h->capture_stream, &g->graph);
    }
    if (e == hipSuccess) e = h->ctx.first_error;
    if (e == hipSuccess) e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      drop_graph(*g);
      h->ctx.first_error = hipSuccess;
      h->use_graphs = false;
      body();                                       // nothing ran during the failed capture
      return finish(h);
    }
  }
  if (hipGraphLaunch(g->exec, h->ctx.stream) != hipSuccess) return fail(h, BETTY_EDEVICE, "hipGraphLaunch failed");
  if (g->replays < 16) ++g->replays;
  return BETTY_OK;
}

static betty_handle_s::CallKey call_key(std::initializer_list<const void*> ptr, int K = -1, std::initializer_list<float> f = {}) {
  betty_handle_s::CallKey key;
  std::copy(ptr.begin(), ptr.end(), key.ptr);
  std::copy(f.begin(), f.end(), key.f);
  key.k[0] = K;
  return key;
}

static betty_status check_hyper_args(betty_handle h, const float* w, const float* lambda, int K, float alpha,
                                     float* dlambda) {
  CHECK(check_ready(h));
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, dlambda, "dlambda"));
  if (K < 0) return fail(h, BETTY_EINVAL, "K must be >= 0 (got %d)", K);
  if (!std::isfinite(alpha)) return fail(h, BETTY_EINVAL, "alpha must be finite");
  if (overlaps(dlambda, h->n_hyper * 4, w, h->d * 4) || overlaps(dlambda, h->n_hyper * 4, lambda, h->n_hyper * 4))
    return fail(h, BETTY_EINVAL, "dlambda overlaps an input");
  return BETTY_OK;
}

// ---- the Neumann series in sample space ----------------------------------------------------------
//
// Without a per-parameter diagonal (reweighting cost; the proximal cost has one constant per layer) the
// Hessian of the batch acts through its samples: per layer H V = Ra^T delta + a^T R delta (+ 2 rho V), and
// what the next product needs of V are only a V and delta V^T.  Both follow from V's own recurrence
// V <- g + beta V - alpha (Ra^T delta + a^T R delta), beta = 1 - 2 alpha rho, through matrices over pairs of
// samples:
//   AS = a V + c          <-  Ag + beta AS - alpha [ (a Ra^T) delta + (a a^T + 1) R delta ]
//   DS = delta V^T        <-  Dg + beta DS - alpha [ (delta R delta^T) a + (delta delta^T) Ra ]
// so no parameter-sized vector is formed, read or written between the steps, the links of the R-op chains
// carry half the reduction (the direction's half is AS, DS), and layer 1 has no link at all (R a_0 = 0).
// Per layer and step 10 B^2 (n_in + n_out) operations with bf16 operands (6 with fp32) take the place of
// 8 B n_in n_out and of the parameter-sized traffic (121M-parameter model, batch 512: 5.88 -> 3.80 ms per
// hypergradient; 2000 x 4 - 700, batch 100: 837 -> 478 us).  AS and DS stay fp32, the operands are those the
// parameter-sized products would take; the matrices over samples are kept as value + remainder with bf16
// operands, since their entries share a large common part whose rounding would not cancel.
struct SampleLaunch {
  betty_handle h;
  OperandSet& os;
  GemmBatch b;
  double flops = 0;
  int mode;
  SampleLaunch(betty_handle h_, OperandSet& os_, int mode_) : h(h_), os(os_), mode(mode_) {}
  GemmProblem& add(int M, int N, int Ktot) {
    if (b.n == MAX_SAMPLE_PROBLEMS) flush();
    GemmProblem& p = b.p[b.n++];
    p.e = blank_epilogue(mode);
    p.g.M = M; p.g.N = N;
    flops += 2.0 * M * N * Ktot;
    return p;
  }
  // C = A B^T + gamma over pairs of samples; A [rows][ld], B [cols][ld]
  void gram(const void* A, int lda, const void* B, int ldb, int rows, int cols, int K, float gamma, size_t out, int ldo) {
    GemmProblem& p = add(rows, cols, K);
    set_pairs(p.g, A, lda, B, ldb, K, nullptr, 0, nullptr, 0, 0);
    p.e.gamma = gamma;
    p.e.out = h->at<void>(out); p.e.ld = ldo;
  }
  void flush() {
    if (b.n == 0) return;
    launch_gemm_batch(h->ctx, os.elem, plan_chain(h, os.elem, b), b, flops);
    b = GemmBatch();
    flops = 0;
  }
};

// what the train side's activations a_{l-1} are called
const void* act_rows(betty_handle h, OperandSet& os, int side, int l) { return l == 1 ? h->at<void>(os.side[side].X) : h->at<void>(os.side[side].A[l - 1]); }
const void* act_cols(betty_handle h, OperandSet& os, int side, int l) { return l == 1 ? h->at<void>(os.side[side].XT) : h->at<void>(os.side[side].At[l - 1]); }

// epilogue of a SAMPLE problem that leaves a V + c (or delta V^T) in `to`; for layer 1 of a deeper network R a_1 too
void sample_sum(betty_handle h, OperandSet& os, GemmProblem& p, size_t to, int ldf, bool first_layer) {
  p.e.f0 = h->f(to);
  p.e.ldf = ldf;
  if (!first_layer || h->L < 2) return;
  p.e.dphi = h->f(os.side[0].dphi[1]);
  p.e.out = h->at<void>(os.RA1); p.e.ld = ldf;
  p.e.outT = h->at<void>(os.RA1t); p.e.ldT = os.side[0].Bp;
}
void next_RA1(OperandSet& os) { std::swap(os.RA[1], os.RA1); std::swap(os.RAt[1], os.RA1t); }

// Ag, Dg from the validation batch (u = grad_w L_U = a_val^T delta_val) or from the dense vector u, and the
// matrices that stay the same over the steps
void samples_begin(betty_handle h, OperandSet& os, const float* u_or_null, bool steps) {
  SideBuf& sb = os.side[0];
  SideBuf& vb = os.side[1];
  const int L = h->L, B = sb.B;
  const float one = h->desc.has_bias ? 1.f : 0.f;
  SampleLaunch gram(h, os, EPI_GRAM);
  for (int l = 1; l <= L; ++l) {
    const LayerInfo& li = h->layers[l - 1];
    const void* a = act_rows(h, os, 0, l);
    const void* D = h->at<void>(sb.D[l]);
    if (!u_or_null) {
      gram.gram(a, li.n_in_p, act_rows(h, os, 1, l), li.n_in_p, B, vb.B, li.n_in, one, os.Gx[l], os.ldGx);
      if (l > 1 && steps) gram.gram(D, li.n_out_p, h->at<void>(vb.D[l]), li.n_out_p, B, vb.B, li.n_out, 0.f, os.Ex[l], os.ldGx);
    }
    if (!steps) continue;
    gram.gram(a, li.n_in_p, a, li.n_in_p, B, B, li.n_in, one, os.G[l], os.ldG);
    if (l > 1) gram.gram(D, li.n_out_p, D, li.n_out_p, B, B, li.n_out, 0.f, os.E[l], os.ldG);
  }
  gram.flush();
  SampleLaunch sum(h, os, EPI_SAMPLE);
  for (int l = 1; l <= L; ++l) {
    const LayerInfo& li = h->layers[l - 1];
    GemmProblem& p = sum.add(B, li.n_out, u_or_null ? li.n_in : vb.B);
    if (u_or_null) {
      set_pairs(p.g, act_rows(h, os, 0, l), li.n_in_p, h->at<void>(os.Vt[l - 1]), li.n_in_p, li.n_in, nullptr, 0, nullptr, 0, 0);
      p.e.colvec = h->desc.has_bias ? u_or_null + li.b_off : nullptr;
    } else {
      set_pairs(p.g, h->at<void>(os.Gx[l]), os.ldGx, h->at<void>(vb.Dt[l]), vb.Bp, vb.B, nullptr, 0, nullptr, 0, 0);
      p.g.split = os.elem == ELEM_BF16;
    }
    p.e.alpha = -1.f;
    sample_sum(h, os, p, os.Ag[l], li.n_out_p, l == 1);
    if (l == 1 || !steps) continue;
    GemmProblem& q = sum.add(B, li.n_in, u_or_null ? li.n_out : vb.B);
    if (u_or_null) {
      set_pairs(q.g, h->at<void>(sb.D[l]), li.n_out_p, h->at<void>(os.Vn[l - 1]), li.n_out_p, li.n_out, nullptr, 0, nullptr, 0, 0);
    } else {
      set_pairs(q.g, h->at<void>(os.Ex[l]), os.ldGx, act_cols(h, os, 1, l), vb.Bp, vb.B, nullptr, 0, nullptr, 0, 0);
      q.g.split = os.elem == ELEM_BF16;
    }
    q.e.alpha = -1.f;
    sample_sum(h, os, q, os.Dg[l], li.n_in_p, false);
  }
  sum.flush();
  if (L >= 2) next_RA1(os);
}

// R-forward links 2 ... upto with a V + c given (in AS, layer 1's Ra_1 with it)
void samples_r_forward(betty_handle h, OperandSet& os, const std::vector<size_t>& AS, int upto) {
  SideBuf& sb = os.side[0];
  for (int l = 2; l <= upto; ++l) {
    const LayerInfo& li = h->layers[l - 1];
    const bool last = l == h->L;
    Epilogue e = blank_epilogue(last ? EPI_RFWD_LAST : EPI_RFWD);
    e.e = h->f(AS[l]);
    e.f0 = h->f(os.Rz[l]);
    e.ldf = li.n_out_p;
    if (!last) {
      e.dphi = h->f(sb.dphi[l]);
      e.out = h->at<void>(os.RA[l]); e.ld = li.n_out_p;
      e.outT = h->at<void>(os.RAt[l]); e.ldT = sb.Bp;
    }
    chain_gemm(h, os.elem, h->at<void>(os.RA[l - 1]), li.n_in_p, h->at<void>(os.Wt[l - 1]), li.n_in_p, li.n_in,
               nullptr, 0, nullptr, 0, 0, sb.B, li.n_out, e, 2.0 * sb.B * li.n_in * li.n_out);
  }
}

// the narrow output layer of the R-op passes with a V + c and delta V^T given
LastRopArgs samples_last_args(betty_handle h, OperandSet& os, const std::vector<size_t>& AS) {
  SideBuf& sb = os.side[0];
  const int L = h->L;
  const LayerInfo& lo = h->layers[L - 1];
  LastRopArgs a{};
  a.RA = h->at<void>(os.RA[L - 1]); a.lda = lo.n_in_p;
  a.Wt = h->at<void>(os.Wt[L - 1]); a.ldt = lo.n_in_p;
  a.Wn = h->at<void>(os.Wn[L - 1]); a.ldn = lo.n_out_p;
  a.AS = h->f(AS[L]); a.ldas = lo.n_out_p;
  a.P = h->f(sb.P); a.ldp = lo.n_out_p;
  a.B = sb.B; a.n_in = lo.n_in; a.C = lo.n_out; a.loss = h->desc.loss;
  return a;
}

// The R-op chains along the current partial sum, and the matrices that its update takes (if one follows).
// `last` (reweighting cost): only a V is needed afterwards, for the mixed term.
void samples_chains(betty_handle h, OperandSet& os, bool first, bool update, bool last) {
  SideBuf& sb = os.side[0];
  const int L = h->L, B = sb.B, Bp = sb.Bp;
  const std::vector<size_t>& AS = first ? os.Ag : os.AS;
  const std::vector<size_t>& DS = first ? os.Dg : os.DS;
  const LayerInfo& lo = h->layers[L - 1];
  const bool narrow = L >= 2 && lo.n_out <= LAST_ROP_MAX_C;
  samples_r_forward(h, os, AS, narrow ? L - 1 : L);
  auto rz = [&](int l) { return h->f(l == 1 ? AS[1] : os.Rz[l]); };
  if (narrow) {
    LastRopArgs a = samples_last_args(h, os, AS);
    a.DS = h->f(DS[L]);
    a.s = h->f(sb.s);
    a.DL = h->at<void>(sb.D[L]); a.ldd = lo.n_out_p;
    a.dphi = h->f(sb.dphi[L - 1]); a.e2 = sb.e2[L - 1] ? h->f(sb.e2[L - 1]) : nullptr;
    a.Rz = rz(L - 1); a.ldf = lo.n_in_p;
    a.RDL = h->at<void>(os.RD[L]); a.RDLt = h->at<void>(os.RDt[L]); a.ldRDLt = Bp;
    a.RD = L > 2 ? h->at<void>(os.RD[L - 1]) : nullptr; a.ldRD = lo.n_in_p; a.RDt = h->at<void>(os.RDt[L - 1]); a.ldRDt = Bp;
    launch_last_layer_rop(h->ctx, os.elem, a);
  } else {
    launch_loss_hessian_rows(h->ctx, os.elem, h->desc.loss, h->f(sb.P), rz(L), lo.n_out_p, h->f(sb.s), B, lo.n_out,
                             h->at<void>(os.RD[L]), lo.n_out_p, h->at<void>(os.RDt[L]), Bp);
  }
  // M and N of the update: ready once their R a and R delta are, so they ride along in the links of the
  // R-backward chain where those leave the chip room, the rest in a launch of their own
  SampleLaunch grams(h, os, EPI_GRAM);
  auto want = [&](int l) {
    const LayerInfo& li = h->layers[l - 1];
    if (!update) return;
    grams.gram(h->at<void>(sb.A[l - 1]), li.n_in_p, h->at<void>(os.RA[l - 1]), li.n_in_p, B, B, li.n_in, 0.f, os.M[l], os.ldG);
    if (!last) grams.gram(h->at<void>(sb.D[l]), li.n_out_p, h->at<void>(os.RD[l]), li.n_out_p, B, B, li.n_out, 0.f, os.N[l], os.ldG);
  };
  if (narrow) want(L);
  for (int l = narrow ? L - 1 : L; l >= 2; --l) {
    want(l);
    const LayerInfo& li = h->layers[l - 1];
    GemmBatch b;
    b.n = 1;
    GemmProblem& p = b.p[0];
    set_pairs(p.g, h->at<void>(os.RD[l]), li.n_out_p, h->at<void>(os.Wn[l - 1]), li.n_out_p, li.n_out, nullptr, 0, nullptr, 0, 0);
    p.g.M = B; p.g.N = li.n_in;
    Epilogue& e = p.e;
    e = blank_epilogue(EPI_RBWD);
    e.e_io = h->f(DS[l]);
    e.dphi = h->f(sb.dphi[l - 1]);
    e.e = sb.e2[l - 1] ? h->f(sb.e2[l - 1]) : nullptr;
    e.Rz = rz(l - 1);
    e.ldf = li.n_in_p;
    e.out = l > 2 ? h->at<void>(os.RD[l - 1]) : nullptr; e.ld = li.n_in_p;
    e.outT = h->at<void>(os.RDt[l - 1]); e.ldT = Bp;
    double flops = 2.0 * B * li.n_in * li.n_out;
    long tiles = Extent::up(B, 32) * Extent::up(li.n_in, 32);
    while (grams.b.n > 0 && b.n < MAX_CHAIN_PROBLEMS) {
      const GemmProblem& g = grams.b.p[grams.b.n - 1];
      tiles += Extent::up(g.g.M, 32) * Extent::up(g.g.N, 32);
      if (tiles > 512) break;
      b.p[b.n++] = g;
      flops += 2.0 * g.g.M * g.g.N * g.g.K[0];
      grams.flops -= 2.0 * g.g.M * g.g.N * g.g.K[0];
      --grams.b.n;
    }
    launch_gemm_batch(h->ctx, os.elem, plan_chain(h, os.elem, b), b, flops);
  }
  grams.flush();
}

// The update of the partial sum after its chains.
void samples_update(betty_handle h, OperandSet& os, bool first, bool last, float alpha) {
  SideBuf& sb = os.side[0];
  const int L = h->L, B = sb.B, Bp = sb.Bp;
  const std::vector<size_t>& AS = first ? os.Ag : os.AS;
  const std::vector<size_t>& DS = first ? os.Dg : os.DS;
  SampleLaunch sum(h, os, EPI_SAMPLE);
  for (int l = 1; l <= L; ++l) {
    const LayerInfo& li = h->layers[l - 1];
    const float beta = (float)series_beta(h, l, alpha);
    GemmProblem& p = sum.add(B, li.n_out, (l == 1 ? 1 : 2) * B);
    if (l == 1) set_pairs(p.g, h->at<void>(os.G[l]), os.ldG, h->at<void>(os.RDt[l]), Bp, B, nullptr, 0, nullptr, 0, 0);
    else set_pairs(p.g, h->at<void>(os.M[l]), os.ldG, h->at<void>(sb.Dt[l]), Bp, B, h->at<void>(os.G[l]), os.ldG,
                   h->at<void>(os.RDt[l]), Bp, B);
    p.g.split = os.elem == ELEM_BF16;
    p.e.alpha = alpha; p.e.beta = beta;
    p.e.e = h->f(AS[l]); p.e.Rz = h->f(os.Ag[l]);
    sample_sum(h, os, p, os.AS[l], li.n_out_p, l == 1);
    if (l == 1 || last) continue;
    GemmProblem& q = sum.add(B, li.n_in, 2 * B);
    set_pairs(q.g, h->at<void>(os.N[l]), os.ldG, act_cols(h, os, 0, l), Bp, B, h->at<void>(os.E[l]), os.ldG,
              h->at<void>(os.RAt[l - 1]), Bp, B);
    q.g.split = os.elem == ELEM_BF16;
    q.e.alpha = alpha; q.e.beta = beta;
    q.e.e = h->f(DS[l]); q.e.Rz = h->f(os.Dg[l]);
    sample_sum(h, os, q, os.DS[l], li.n_in_p, false);
  }
  sum.flush();
  if (L >= 2) next_RA1(os);
}

// Proximal cost: sum_k beta^(K-1-k) (Ra, R delta) of the steps, in fp32.  As operands of the final product it stands in
// RAt, RDt (fp32) or as value and remainder in sumRA, sumRD (bf16: rounding the sum once more would cost the last step
// as much precision as all the products before; 2^-9 of it stays 2^-18 this way).
void samples_accumulate(betty_handle h, OperandSet& os, bool first, bool last, float alpha) {
  const size_t Bp = os.side[0].Bp;
  AccumulateBatch b;
  b.first = first; b.last = last;
  auto add = [&](size_t r, size_t sum, float beta, int rows) {
    if (b.n == MAX_PROBLEMS) { launch_accumulate(h->ctx, os.elem, b); b.n = 0; }
    b.j[b.n++] = AccumulateJob{h->at<void>(r), h->f(sum), beta, rows * Bp};
  };
  for (int l = 1; l <= h->L; ++l) {
    add(os.RDt[l], os.sumRD[l], (float)series_beta(h, l, alpha), h->layers[l - 1].n_out_p);
    if (l < h->L) add(os.RAt[l], os.sumRA[l], (float)series_beta(h, l + 1, alpha), h->layers[l - 1].n_out_p);
  }
  launch_accumulate(h->ctx, os.elem, b);
}

void neumann_samples_seq(betty_handle h, const float* w, const float* lambda, const float* u_or_null, int K, float alpha,
                         float* out) {
  OperandSet& os = h->sets[0];
  const bool rw = h->desc.hp == BETTY_HP_REWEIGHT_NET;
  const int L = h->L;
  const LayerInfo& lo = h->layers[L - 1];
  // (the two places of R a_1 trade names; a product that is asked for later finds the one it knows)
  struct Home {
    OperandSet& os;
    const size_t ra;
    ~Home() { if (os.RA[1] != ra) next_RA1(os); }
  } home{os, os.RA[1]};
  make_weight_operands(h, os, w, u_or_null);
  if (u_or_null) {
    prepare_lower(h, os, w, lambda);
  } else {
    const Pass ps[2] = {train_pass(h, os, w, lambda, true), val_pass(os, w)};
    forward_backward(h, ps, 2);
  }
  samples_begin(h, os, u_or_null, K > 0);
  for (int k = 0; k < K; ++k) {
    const bool last = k + 1 == K;
    const bool update = rw || !last;
    samples_chains(h, os, k == 0, update, last);
    if (!rw && K > 1) samples_accumulate(h, os, k == 0, last, alpha);
    if (update) samples_update(h, os, k == 0, last, alpha);
  }
  SideBuf& sb = os.side[0];
  if (rw) {
    // the mixed term is one more R-forward along the final sum
    const std::vector<size_t>& AS = K > 0 ? os.AS : os.Ag;
    const bool narrow = L >= 2 && lo.n_out <= LAST_ROP_MAX_C;
    samples_r_forward(h, os, AS, narrow ? L - 1 : L);
    if (narrow) {
      LastRopArgs a = samples_last_args(h, os, AS);
      a.cvec = h->f(os.cvec); a.labels = h->at<Labels>(h->labels); a.Z = h->f(sb.ZL);
      launch_last_layer_rop(h->ctx, os.elem, a);
    } else {
      launch_loss_directional_rows(h->ctx, h->desc.loss, h->f(sb.P), h->f(sb.ZL), h->at<Labels>(h->labels),
                                   h->f(L == 1 ? AS[1] : os.Rz[L]), lo.n_out_p, sb.B, lo.n_out, h->f(os.cvec));
    }
    launch_wnet_theta_vjp(h->ctx, h->f(sb.ell), h->f(sb.dsig), h->f(os.cvec), nullptr, nullptr, lambda, h->desc.wnet_hidden,
                          sb.B, alpha / (float)sb.B, out);
    return;
  }
  // proximal cost: d(anchor) = 2 rho alpha s with s = (sum_j beta^j) g - alpha sum_k beta^(K-1-k) (Ra^T delta + a^T R delta)_k
  const float* g = u_or_null;
  if (!g) {
    wgrad_batch(h, os, 1, false, WgradSink{EPI_WGRAD, h->f(h->vec_v), nullptr, nullptr, nullptr, nullptr, 0.f, false});
    g = h->f(h->vec_v);
  }
  WgradSink fin{EPI_WGRAD_SCALED, out, nullptr, g, nullptr, nullptr, alpha, false};
  fin.K = K;
  fin.sums_split = os.elem == ELEM_BF16 && K > 1;
  wgrad_batch(h, os, 0, true, fin);
}

void linear_seq(betty_handle h, const float* w, const float* lambda, int K, float alpha, float* out, bool cg) {
  const LayerInfo& li = h->layers[0];
  LinearArgs a{};
  for (int s = 0; s < 2; ++s) {
    const SideBuf& sb = h->sets[0].side[s];
    a.X[s] = h->f(sb.X); a.XT[s] = h->f(sb.XT); a.ldxt[s] = sb.Bp; a.B[s] = sb.B;
  }
  a.ldx = li.n_in_p; a.n_in = li.n_in; a.C = li.n_out; a.bias = h->desc.has_bias ? 1 : 0;
  a.labels = h->at<Labels>(h->labels); a.loss = h->desc.loss;
  a.K = K; a.alpha = alpha; a.w = w; a.lam = lambda; a.out = out;
  if (h->desc.loss == BETTY_LOSS_MSE && !cg) a.G = h->f(h->lin_gram);
  launch_linear_hypergrad(h->ctx, a, cg);
}

// out = (dw* / dlambda) u by the K-step Neumann series and the mixed VJP; u = grad_w L_U(w) on the
// validation batch when u_or_null is null.  Only enqueues launches on the handle's stream.
// The partial sum is carried in nested form, s <- g + (I - alpha H) s from s = g: after K steps
// s = sum_{j<=K} (I - alpha H)^j g, with one parameter-sized state vector to read and write per step.
static void neumann_seq(betty_handle h, const float* w, const float* lambda, const float* u_or_null, int K,
                        float alpha, float* out) {
  if (use_samples(h, K, u_or_null != nullptr)) {
    neumann_samples_seq(h, w, lambda, u_or_null, K, alpha, out);
    return;
  }
  OperandSet& os = h->sets[0];
  const bool l2 = h->desc.hp == BETTY_HP_L2_DECAY, rw = h->desc.hp == BETTY_HP_REWEIGHT_NET;
  const float* dl = diag_log(h, lambda);
  float* s = h->f(h->vec_p);
  const float* g = u_or_null;
  const bool need_lower = K > 0 || rw;      // forward/backward cache of the train batch
  make_weight_operands(h, os, w, K > 0 || rw ? u_or_null : nullptr);
  // the reweighting mixed term runs one more R-forward along the final sum: its operand copies are
  // written by whichever launch produces that sum
  if (u_or_null) {
    if (need_lower) prepare_lower(h, os, w, lambda);
  } else {
    // g = grad_w L_U lands in vec_v, with its operand copies for the first product
    WgradSink init{EPI_WGRAD_INIT, nullptr, nullptr, nullptr, h->f(h->vec_v), nullptr, 0.f, K > 0 || rw};
    upper_grad_seq(h, os, w, lambda, need_lower, init, nullptr);
    g = h->f(h->vec_v);
  }
  const float* s_cur = g;                   // s_0 = g
  for (int k = 0; k < K; ++k) {
    // the step is fused into the weight-gradient epilogues of the product; for L2 decay the last
    // step also applies the mixed VJP, so only d(lambda) is written.
    // With the second stream, layer l's launch runs while the R-backward chain is still reading
    // this product's direction copies of the layers below, so the new copies go to the other set.
    const bool last = k + 1 == K;
    const bool pipe = h->use_pipeline && h->side_stream && h->L >= 2;
    if (last && l2) {
      WgradSink fin{EPI_WGRAD_NEUMANN_L2, out, lambda, w, const_cast<float*>(g), const_cast<float*>(s_cur), alpha, false};
      hvp_cached(h, os, s_cur, fin, pipe);
    } else {
      WgradSink step{EPI_WGRAD_NEUMANN, nullptr, dl, s_cur, const_cast<float*>(g), s, alpha, !last || rw};
      step.second_set = pipe;
      hvp_cached(h, os, s_cur, step, pipe);
      if (pipe && step.copies) { std::swap(os.Vn, os.Vn2); std::swap(os.Vt, os.Vt2); }
    }
    s_cur = s;
  }
  if (l2) {
    if (K == 0) launch_mixed_l2(h->ctx, lambda, w, s_cur, alpha, out, h->d);
  } else if (rw) {
    mixed_reweight_seq(h, os, lambda, s_cur, alpha, out, true);
  } else {
    launch_mixed_prox(h->ctx, h->f(h->logrho), s_cur, alpha, out, h->d);
  }
}

extern "C" {

betty_status betty_create(const betty_problem_desc* desc, betty_handle* out) {
  if (!desc || !out) return BETTY_ENULL;
  *out = nullptr;
  if (!desc->dims) return BETTY_ENULL;
  if (desc->n_layers < 1 || desc->n_layers > 64) return BETTY_ESHAPE;
  for (int i = 0; i <= desc->n_layers; ++i)
    if (desc->dims[i] < 1 || desc->dims[i] > (1 << 20)) return BETTY_ESHAPE;
  if (desc->batch_train < 1 || desc->batch_val < 1 || desc->batch_train > (1 << 20) || desc->batch_val > (1 << 20))
    return BETTY_ESHAPE;
  if (desc->act < BETTY_ACT_NONE || desc->act > BETTY_ACT_GELU_ERF) return BETTY_EINVAL;
  if (desc->loss != BETTY_LOSS_MSE && desc->loss != BETTY_LOSS_SOFTMAX_CE) return BETTY_EINVAL;
  if (desc->hp != BETTY_HP_L2_DECAY && desc->hp != BETTY_HP_REWEIGHT_NET && desc->hp != BETTY_HP_PROXIMAL)
    return BETTY_EINVAL;
  if (desc->hp == BETTY_HP_PROXIMAL && !(std::isfinite(desc->prox_rho) && desc->prox_rho >= 0.f)) return BETTY_EINVAL;
  if (desc->prec != BETTY_PREC_FP32 && desc->prec != BETTY_PREC_BF16_FP32ACC) return BETTY_EINVAL;
  if (desc->hp == BETTY_HP_REWEIGHT_NET && (desc->wnet_hidden < 1 || desc->wnet_hidden > 65536)) return BETTY_ESHAPE;

  // the kernels index one matrix (a layer's weights, an activation) with 32-bit offsets
  {
    const long long bp = padup(std::max(desc->batch_train, desc->batch_val));
    for (int i = 0; i < desc->n_layers; ++i) {
      const long long a = padup(desc->dims[i]), b = padup(desc->dims[i + 1]);
      if (a * b >= (1LL << 31) || bp * a >= (1LL << 31) || bp * b >= (1LL << 31)) return BETTY_ESHAPE;
    }
  }

  betty_handle h = new (std::nothrow) betty_handle_s();
  if (!h) return BETTY_EDEVICE;
  h->desc = *desc;
  h->dims.assign(desc->dims, desc->dims + desc->n_layers + 1);
  h->desc.dims = h->dims.data();
  h->L = desc->n_layers;
  size_t off = 0;
  for (int l = 0; l < h->L; ++l) {
    LayerInfo li{};
    li.n_in = h->dims[l]; li.n_out = h->dims[l + 1];
    li.n_in_p = padup(li.n_in); li.n_out_p = padup(li.n_out);
    li.w_off = off; off += (size_t)li.n_in * li.n_out;
    li.b_off = off;
    if (desc->has_bias) off += li.n_out;
    h->layers.push_back(li);
    h->max_np = std::max(h->max_np, std::max(li.n_in_p, li.n_out_p));
  }
  h->d = off;
  h->n_hyper = desc->hp == BETTY_HP_REWEIGHT_NET ? (size_t)3 * desc->wnet_hidden + 1 : h->d;
  // Large models with fp32 operands overlap each layer's weight-gradient launch with the R-backward
  // chain (see use_pipeline).  With bf16 operands their weight gradients take the 128-tile kernel,
  // all layers in one launch behind the chain: measured on the 121M-parameter model, 7.23 ms per
  // hypergradient against 7.49 ms for the overlapped 64-tile launches and 8.37 ms for overlapped
  // 128-tile ones (the two streams contend for the same memory path).
  const bool large = h->d >= ((size_t)32 << 20);
  h->use_pipeline = large && desc->prec == BETTY_PREC_FP32;
  h->fd_paired = !large;
  h->max_Bp = std::max(padup(desc->batch_train), padup(desc->batch_val));
  // tuning overrides for experiments: BETTY_TUNE="wgrad=<cfg>,wgrad128=<n>,tile128=<n>,blocks=1,pair=1,rect=<n>,pipe=<0|1>,fd2=<0|1>,samples=<0|1>,linear=<0|1>,narrow=<0..4>,layer1=<0|1>" (see plan_chain)
  if (const char* t = getenv("BETTY_TUNE")) {
    int v;
    if (const char* q = strstr(t, "wgrad=")) if (sscanf(q + 6, "%d", &v) == 1 && (v == GEMM_128x1 || v == GEMM_64x1)) h->tune_wgrad_cfg = v;
    if (const char* q = strstr(t, "tile128=")) if (sscanf(q + 8, "%d", &v) == 1 && v > 0) h->tune_tile128_min = v;
    // blocks=1: no K-split kernel; rect above 1024: 128 x 64 tiles wherever 128-tiles are not taken
    if (const char* q = strstr(t, "blocks=")) if (sscanf(q + 7, "%d", &v) == 1) h->tune_split = v != 1;
    if (const char* q = strstr(t, "rect=")) if (sscanf(q + 5, "%d", &v) == 1) h->tune_rect_forced = v > 1024;
    if (const char* q = strstr(t, "wgrad128=")) if (sscanf(q + 9, "%d", &v) == 1 && v >= 0) h->tune_wgrad128_min = v;
    if (const char* q = strstr(t, "pipe=")) if (sscanf(q + 5, "%d", &v) == 1) h->use_pipeline = v != 0;
    if (const char* q = strstr(t, "samples=")) if (sscanf(q + 8, "%d", &v) == 1) h->tune_samples = v != 0;
    if (const char* q = strstr(t, "pair=")) if (sscanf(q + 5, "%d", &v) == 1) h->tune_pair_forced = v == 1;
    if (const char* q = strstr(t, "narrow=")) if (sscanf(q + 7, "%d", &v) == 1 && v >= 0 && v <= 4) h->tune_narrow = v;
    if (const char* q = strstr(t, "layer1=")) if (sscanf(q + 7, "%d", &v) == 1) h->tune_layer1 = v != 0;
    if (const char* q = strstr(t, "linear=")) if (sscanf(q + 7, "%d", &v) == 1) h->tune_linear = v != 0;
    if (const char* q = strstr(t, "fd2=")) if (sscanf(q + 4, "%d", &v) == 1) h->fd_paired = v != 0;
  }
  plan(h);
  *out = h;
  return BETTY_OK;
}

void betty_destroy(betty_handle h) {
  if (!h) return;
  drop_graphs(h);
  release_side_stream(h);
  if (h->capture_stream) (void)hipStreamDestroy(h->capture_stream);
  if (h->order_event) (void)hipEventDestroy(h->order_event);
  for (auto& r : h->ctx.recs) { (void)hipEventDestroy(r.e0); (void)hipEventDestroy(r.e1); }
  delete h;
}

const char* betty_last_error(betty_handle h) { return h ? h->err.c_str() : "null handle"; }
size_t betty_num_params(betty_handle h) { return h ? h->d : 0; }
size_t betty_num_hyper(betty_handle h) { return h ? h->n_hyper : 0; }
size_t betty_workspace_bytes(betty_handle h) { return h ? h->ws_need : 0; }

betty_status betty_bind(betty_handle h, void* workspace, size_t bytes, void* hip_stream) {
  if (!h) return BETTY_ENULL;
  if (!workspace) return fail(h, BETTY_ENULL, "workspace is NULL");
  if (((uintptr_t)workspace) & 255) return fail(h, BETTY_EALIGN, "workspace is not 256-byte aligned");
  if (bytes < h->ws_need) return fail(h, BETTY_EWORKSPACE, "workspace has %zu bytes, %zu needed", bytes, h->ws_need);
  h->ws = (char*)workspace;
  h->ctx.stream = h->bound_stream = (hipStream_t)hip_stream;
  if (!h->side_stream && hip_stream != nullptr) {
    // second stream (default priority) and the events that order it against the bound stream
    bool ok = hipStreamCreateWithFlags(&h->side_stream, hipStreamNonBlocking) == hipSuccess;
    h->fork_events.assign(h->L, nullptr);
    for (int l = 0; ok && l < h->L; ++l)
      ok = hipEventCreateWithFlags(&h->fork_events[l], hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&h->join_event, hipEventDisableTiming) == hipSuccess;
    if (!ok) { (void)hipGetLastError(); release_side_stream(h); }
  }
  drop_graphs(h);
  h->epoch = next_epoch();
  h->bound = true;
  h->batches = false;
  init_workspace(h, h->ws_need);
  return finish(h);
}

betty_status betty_run_on(betty_handle h, void* hip_stream) {
  if (!h) return BETTY_ENULL;
  if (!h->bound) return BETTY_OK;
  const hipError_t e = move_to_stream(h, (hipStream_t)hip_stream);
  return e == hipSuccess ? BETTY_OK : fail(h, BETTY_EDEVICE, "HIP error: %s", hipGetErrorString(e));
}

// X of the first n batches (train, validation) into every operand set that reads it, and the places of
// the labels, in one launch
static void convert_inputs(betty_handle h, const betty_batch* b, int n) {
  const LayerInfo& l0 = h->layers[0];
  ConvertBatch cb;
  cb.n = n;
  for (int s = 0; s < n; ++s) {
    const SideBuf& sb = h->sets[0].side[s];
    cb.j[s] = ConvertJob{b[s].x, l0.n_in, sb.B, l0.n_in, h->at<void>(sb.X), l0.n_in_p, h->at<void>(sb.XT), sb.Bp};
    if (h->sets[1].present) {
      cb.j[s].out32 = h->f(h->sets[1].side[s].X);
      cb.j[s].outT32 = h->f(h->sets[1].side[s].XT);
    }
  }
  cb.table = h->at<Labels>(h->labels);
  for (int s = 0; s < 2; ++s) cb.labels[s] = Labels{b[s < n ? s : 0].y, b[s < n ? s : 0].target};
  launch_convert_batch(h->ctx, h->sets[0].elem, cb);
}

betty_status betty_set_batches(betty_handle h, betty_batch train, betty_batch val) {
  if (!h) return BETTY_ENULL;
  if (!h->bound) return fail(h, BETTY_EWORKSPACE, "no workspace bound (call betty_bind)");
  const betty_batch b[2] = {train, val};
  for (int s = 0; s < 2; ++s) {
    CHECK(check_vec(h, b[s].x, s ? "val.x" : "train.x"));
    if (h->desc.loss == BETTY_LOSS_SOFTMAX_CE) CHECK(check_vec(h, b[s].y, s ? "val.y" : "train.y"));
    else CHECK(check_vec(h, b[s].target, s ? "val.target" : "train.target"));
  }
  convert_inputs(h, b, 2);
  h->batches = true;
  return finish(h);
}

betty_status betty_lower_grad(betty_handle h, const float* w, const float* lambda, float* grad_w,
                              float* loss_or_null) {
  CHECK(check_ready(h));
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, grad_w, "grad_w"));
  if (loss_or_null) CHECK(check_vec(h, loss_or_null, "loss"));
  if (overlaps(grad_w, h->d * 4, w, h->d * 4) || overlaps(grad_w, h->d * 4, lambda, h->n_hyper * 4))
    return fail(h, BETTY_EINVAL, "grad_w overlaps an input");
  return run_cached(h, h->CALL_LOWER, call_key({w, lambda, grad_w, loss_or_null}), [=]() {
    OperandSet& os = h->sets[0];
    make_weight_operands(h, os, w);
    lower_grad_seq(h, os, w, lambda, grad_w, loss_or_null);
  });
}

betty_status betty_upper_grad(betty_handle h, const float* w, float* grad_w, float* loss_or_null) {
  CHECK(check_ready(h));
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, grad_w, "grad_w"));
  if (loss_or_null) CHECK(check_vec(h, loss_or_null, "loss"));
  if (overlaps(grad_w, h->d * 4, w, h->d * 4)) return fail(h, BETTY_EINVAL, "grad_w overlaps w");
  return run_cached(h, h->CALL_UPPER, call_key({w, grad_w, loss_or_null}), [=]() {
    OperandSet& os = h->sets[0];
    make_weight_operands(h, os, w);
    WgradSink k{EPI_WGRAD, grad_w, nullptr, nullptr, nullptr, nullptr, 0.f, false};
    upper_grad_seq(h, os, w, nullptr, false, k, loss_or_null);
  });
}

static betty_status check_hvp_args(betty_handle h, const float* w, const float* lambda, const float* v, float* Hv) {
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, v, "v"));
  CHECK(check_vec(h, Hv, "Hv"));
  if (overlaps(Hv, h->d * 4, w, h->d * 4) || overlaps(Hv, h->d * 4, v, h->d * 4) ||
      overlaps(Hv, h->d * 4, lambda, h->n_hyper * 4))
    return fail(h, BETTY_EINVAL, "Hv overlaps an input");
  return BETTY_OK;
}

// one stand-alone Hessian-vector product: operand copies of w, the forward/backward cache of the
// train batch, operand copies of v, the forward-over-reverse passes
static void hvp_seq(betty_handle h, const float* w, const float* lambda, const float* v, float* Hv) {
  OperandSet& os = h->sets[0];
  make_weight_operands(h, os, w, v);
  prepare_lower(h, os, w, lambda);
  const float* dl = diag_log(h, lambda);
  WgradSink k{EPI_WGRAD, Hv, dl, dl ? v : nullptr, nullptr, nullptr, 0.f, false};
  hvp_cached(h, os, v, k);
}

betty_status betty_hvp(betty_handle h, const float* w, const float* lambda, const float* v, float* Hv) {
  CHECK(check_ready(h));
  CHECK(check_hvp_args(h, w, lambda, v, Hv));
  return run_cached(h, h->CALL_HVP, call_key({w, lambda, v, Hv}), [=]() { hvp_seq(h, w, lambda, v, Hv); });
}

// ---- the same product for callers that cannot allocate device memory ----------------------
// The workspace is a fixed array in the library's device image; every GPU the library runs on has
// its own copy at its own address, looked up once per device.
static __device__ __align__(256) unsigned char scratch[BETTY_STATIC_SCRATCH_BYTES];

static betty_status static_scratch(betty_handle h, char** out) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static char* base[MAX_DEVICES] = {};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES)
    return fail(h, BETTY_EDEVICE, "no current HIP device (or its index is beyond %d)", MAX_DEVICES - 1);
  std::lock_guard<std::mutex> lock(mu);
  if (!base[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(h, BETTY_EDEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    base[dev] = (char*)p;
  }
  *out = base[dev];
  return BETTY_OK;
}

size_t betty_static_scratch_bytes(void) { return BETTY_STATIC_SCRATCH_BYTES; }

betty_status betty_hvp_static(betty_handle h, betty_batch train, void* hip_stream, const float* w,
                              const float* lambda, const float* v, float* Hv) {
  if (!h) return BETTY_ENULL;
  CHECK(check_hvp_args(h, w, lambda, v, Hv));
  CHECK(check_vec(h, train.x, "train.x"));
  if (h->desc.loss == BETTY_LOSS_SOFTMAX_CE) CHECK(check_vec(h, train.y, "train.y"));
  else CHECK(check_vec(h, train.target, "train.target"));
  if (h->ws_product > BETTY_STATIC_SCRATCH_BYTES)
    return fail(h, BETTY_EWORKSPACE, "this problem needs %zu bytes of workspace, the library's fixed scratch array holds %zu: "
                "use betty_bind with a caller-owned workspace and betty_hvp", h->ws_product, (size_t)BETTY_STATIC_SCRATCH_BYTES);
  char* base = nullptr;
  CHECK(static_scratch(h, &base));
  // run on the scratch array and the given stream, with the handle's own binding set aside
  char* const ws0 = h->ws;
  const hipStream_t st0 = h->ctx.stream;
  const bool prof0 = h->ctx.profiling;
  h->ws = base;
  h->ctx.stream = (hipStream_t)hip_stream;
  h->ctx.profiling = false;                         // (event creation allocates)
  init_workspace(h, h->ws_product);                 // the array keeps the last call's contents
  convert_inputs(h, &train, 1);
  hvp_seq(h, w, lambda, v, Hv);
  h->ws = ws0;
  h->ctx.stream = st0;
  h->ctx.profiling = prof0;
  return finish(h);
}

betty_status betty_mixed_vjp(betty_handle h, const float* w, const float* lambda, const float* q, float* out) {
  CHECK(check_ready(h));
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, q, "q"));
  CHECK(check_vec(h, out, "out"));
  if (overlaps(out, h->n_hyper * 4, w, h->d * 4) || overlaps(out, h->n_hyper * 4, q, h->d * 4) ||
      overlaps(out, h->n_hyper * 4, lambda, h->n_hyper * 4))
    return fail(h, BETTY_EINVAL, "out overlaps an input");
  if (h->desc.hp == BETTY_HP_L2_DECAY) {
    launch_mixed_l2(h->ctx, lambda, w, q, 1.f, out, h->d);
    return finish(h);
  }
  if (h->desc.hp == BETTY_HP_PROXIMAL) {
    launch_mixed_prox(h->ctx, h->f(h->logrho), q, 1.f, out, h->d);
    return finish(h);
  }
  return run_cached(h, h->CALL_MIXED, call_key({w, lambda, q, out}), [=]() {
    OperandSet& os = h->sets[0];
    make_weight_operands(h, os, w, q, true);
    const Pass ps = train_pass(h, os, w, lambda, false);
    forward_and_loss(h, &ps, 1);
    mixed_reweight_seq(h, os, lambda, q, 1.f, out, true);
  });
}

betty_status betty_hypergrad_neumann(betty_handle h, const float* w, const float* lambda, int K, float alpha,
                                     float* dlambda) {
  CHECK(check_hyper_args(h, w, lambda, K, alpha, dlambda));
  if (use_linear(h, false, K)) { linear_seq(h, w, lambda, K, alpha, dlambda, false); return finish(h); }
  auto body = [=]() { neumann_seq(h, w, lambda, nullptr, K, alpha, dlambda); };
  return run_cached(h, h->CALL_NEUMANN, call_key({w, lambda, dlambda}, K, {alpha}), body);
}

betty_status betty_best_response_neumann(betty_handle h, const float* w, const float* lambda, const float* u, int K,
                                         float alpha, float* out) {
  CHECK(check_hyper_args(h, w, lambda, K, alpha, out));
  CHECK(check_vec(h, u, "u"));
  if (overlaps(out, h->n_hyper * 4, u, h->d * 4)) return fail(h, BETTY_EINVAL, "out overlaps u");
  auto body = [=]() { neumann_seq(h, w, lambda, u, K, alpha, out); };
  return run_cached(h, h->CALL_BEST_RESPONSE, call_key({w, lambda, u, out}, K, {alpha}), body);
}

betty_status betty_hypergrad_chain3(betty_handle hp, betty_handle hf, const float* w, const float* theta,
                                    const float* v, int K_pre, float alpha_pre, int K_ft, float alpha_ft,
                                    float* dtheta) {
  if (!hp || !hf) return BETTY_ENULL;
  CHECK(check_hyper_args(hp, w, theta, K_pre, alpha_pre, dtheta));
  if (check_ready(hf) != BETTY_OK) return fail(hp, BETTY_EWORKSPACE, "finetune handle: %s", hf->err.c_str());
  if (hf->desc.hp != BETTY_HP_PROXIMAL) return fail(hp, BETTY_EINVAL, "the finetune handle must be BETTY_HP_PROXIMAL");
  if (hf->d != hp->d) return fail(hp, BETTY_ESHAPE, "finetune handle has %zu parameters, pretrain handle %zu", hf->d, hp->d);
  if (hf->bound_stream != hp->bound_stream) return fail(hp, BETTY_EINVAL, "both handles must be bound to the same stream");
  CHECK(check_vec(hp, v, "v"));
  if (K_ft < 0) return fail(hp, BETTY_EINVAL, "K_finetune must be >= 0 (got %d)", K_ft);
  if (!std::isfinite(alpha_ft)) return fail(hp, BETTY_EINVAL, "alpha_finetune must be finite");
  if (overlaps(dtheta, hp->n_hyper * 4, v, hp->d * 4)) return fail(hp, BETTY_EINVAL, "dtheta overlaps v");
  // rightmost factor first: u = (dv* / dw) grad_v L_U(v) on the finetuning problem (anchor w),
  // kept in that handle's workspace; then (dw* / dtheta) u on the pretraining problem
  if (hf->ctx.profiling) return fail(hp, BETTY_EINVAL, "switch per-launch timing off on the finetune handle first");
  const hipStream_t home = hf->ctx.stream;
  if (const hipError_t e = move_to_stream(hf, hp->ctx.stream); e != hipSuccess)
    return fail(hp, BETTY_EDEVICE, "HIP error: %s", hipGetErrorString(e));
  auto body = [=]() {
    float* u = hf->f(hf->vec_g);
    const hipStream_t own = hf->ctx.stream;
    hf->ctx.stream = hp->ctx.stream;                  // (the recording stream while the sequence is captured)
    neumann_seq(hf, v, w, nullptr, K_ft, alpha_ft, u);
    hf->ctx.stream = own;
    if (hf->ctx.first_error != hipSuccess) {          // reported through the pretrain handle
      if (hp->ctx.first_error == hipSuccess) hp->ctx.first_error = hf->ctx.first_error;
      hf->ctx.first_error = hipSuccess;
    }
    neumann_seq(hp, w, theta, u, K_pre, alpha_pre, dtheta);
  };
  // repeated identical calls replay one captured graph that spans both handles; the finetune handle's
  // workspace is part of what the graph has recorded, so its binding is part of the key
  auto key = call_key({w, theta, v, dtheta, hf}, K_pre, {alpha_pre, alpha_ft});
  key.k[1] = K_ft;
  key.other_epoch = hf->epoch;
  const betty_status st = run_cached(hp, hp->CALL_CHAIN, key, body);
  if (hf->ctx.stream == home) return st;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(hf->ctx.stream, &cap) != hipSuccess) (void)hipGetLastError();
  if (cap != hipStreamCaptureStatusNone) {            // the caller records a graph: its other stream is not drawn in
    hf->ctx.stream = home;
    return st;
  }
  if (const hipError_t e = move_to_stream(hf, home); e != hipSuccess && st == BETTY_OK)
    return fail(hp, BETTY_EDEVICE, "HIP error: %s", hipGetErrorString(e));
  return st;
}

// The two points w +- eps q, q = scale v, as operands: both at once, or the one of `signs` (1 = plus, 2 = minus).
// (layer1: as the others; otherwise its place for W_1^T takes the direction's V_1^T, or nothing where signs = 2)
static void make_perturbed_operands(betty_handle h, const float* w, const float* v, float* eps, float scale, int signs,
                                    int sums, float eps_scale, bool layer1) {
  OperandSet* os[2] = {&fd_operands(h), &h->fd_minus};
  for (int i0 = !layer1 && signs == 2 ? 1 : 0; i0 < h->L; i0 += MAX_PROBLEMS) {
    PerturbBatch b;
    b.n = std::min(MAX_PROBLEMS, h->L - i0);
    b.eps = sums ? nullptr : eps; b.scale = scale; b.signs = signs;
    b.partial = h->at<double>(h->sums); b.n_partial = sums; b.eps_scale = eps_scale; b.eps_out = eps;
    for (int k = 0; k < b.n; ++k) {
      const LayerInfo& li = h->layers[i0 + k];
      PerturbJob& j = b.j[k];
      j = PerturbJob{};
      j.w = w + li.w_off; j.v = v + li.w_off; j.rows = li.n_in; j.cols = li.n_out;
      j.ld = li.n_out_p; j.ldT = li.n_in_p;
      if (!layer1 && i0 + k == 0) { j.w = nullptr; j.outT[0] = h->f(os[0]->Wt[0]); continue; }
      if (h->desc.has_bias) { j.b = w + li.b_off; j.bv = v + li.b_off; }
      for (int s = 0; s < 2; ++s) {
        j.out[s] = i0 + k > 0 ? h->f(os[s]->Wn[i0 + k]) : nullptr; j.outT[s] = h->f(os[s]->Wt[i0 + k]);
        if (h->desc.has_bias) j.bout[s] = h->f(h->bias_pm[s]) + li.b_off;
      }
    }
    launch_perturb(h->ctx, b);
  }
}

// Central differences of first-order passes, fp32 operands throughout.  Both perturbed points go through the
// same launches (or, on large models, one after the other); the deltas of the minus point carry the
// opposite sign, so one weight-gradient launch over both forms the difference of the data terms in its
// accumulators and its epilogue takes the step.  The diagonal terms are linear in w: their differences are
// formed exactly, 2 exp(lambda) v and, in the mixed VJP, -2 exp(lambda) w q.
static void fd_seq(betty_handle h, const float* w, const float* lambda, int K, float alpha, float eps_scale, float* dlambda) {
  OperandSet& os = fd_operands(h);
  OperandSet& om = h->fd_minus;
  SideBuf& sb = os.side[0];
  const bool l2 = h->desc.hp == BETTY_HP_L2_DECAY, rw = h->desc.hp == BETTY_HP_REWEIGHT_NET;
  const float* dl = diag_log(h, lambda);
  float* v = h->f(h->vec_v); float* p = h->f(h->vec_p); float* eps = h->f(h->scalars) + 1;
  int sums = 0;
  make_weight_operands(h, os, w);
  // Layer 1 is linear in the perturbation: z_1 at w +- eps v is X W_1 + b_1 +- eps (X V_1 + c_1).  The first term is
  // formed once, the second once for both points, and neither point needs operand copies of its first layer: half the
  // products of the largest layer and most of the perturbation's traffic (5.3M parameters, 5 differences: 1260 -> 1105 us).
  // z_1 is written once and read at every difference, and but for reweighting, whose pass at w goes over the train batch
  // anyway, it is a product more, the only one that a single difference would save.  So from 128 inputs and 2^25
  // multiplications of that layer for reweighting, and from three differences and 2^28 otherwise: of 1674 calls timed in both
  // forms 302, 4.4 % faster, 10 of them more than 1.5 % slower, at most 2.6 % (with two differences 7 of 27 are slower, up to
  // 8 %).  (At any size: 15-1200-86, batch 976, K = 1 104 -> 124 us.)
  // (Not where a narrow model's first-order pass starts at layer 1: the one at w, which reweighting never takes so, or
  // those at the points.)
  const LayerInfo& l1 = h->layers[0];
  const double products = (double)sb.B * l1.n_in * l1.n_out;
  const bool shared = h->tune_layer1 >= 0 ? h->tune_layer1 == 1
                                          : l1.n_in >= 128 && (rw ? products >= 33554432.0 : K > 2 && products >= 268435456.0);
  auto from_inputs = [&](int samples) { return narrow_first(h, false, ELEM_F32, samples) == 1; };
  const bool split = shared && h->L >= 2 && (K > 0 || rw) && (rw || !from_inputs(h->desc.batch_val)) && !from_inputs(2 * sb.B);
  const Pass at_w = train_pass(h, os, w, lambda, false);
  h->z1_pass = split ? &at_w : nullptr;
  WgradSink init{EPI_WGRAD_INIT, nullptr, nullptr, nullptr, v, K > 0 ? p : nullptr, 0.f, false};
  if (K > 0 || rw) init.sums = &sums;
  const float* omega_bar = nullptr;
  if (!rw) {
    upper_grad_seq(h, os, w, nullptr, false, init, nullptr);
  } else {
    // the reweighting cost holds its sample weights constant in w: evaluate them (and the loss fed
    // to the weight net) once at the unperturbed w and keep them for every perturbed pass
    Pass ps[2] = {train_pass(h, os, w, lambda, false), val_pass(os, w)};
    ps[0].ell = sb.ell_bar; ps[0].omega = sb.omega_bar; ps[0].dsig = sb.dsig_bar;
    forward_and_loss(h, ps, 2);
    backward_chain(h, ps + 1, 1);
    wgrad_batch(h, os, 1, false, init);
    omega_bar = h->f(sb.omega_bar);
  }
  h->z1_pass = nullptr;
  auto first_layer = [&](const float* dir, float scale) {
    SideBuf& mb = om.side[0];
    Epilogue e = blank_epilogue(EPI_FWD_PM, h->desc.act);
    e.colvec = h->desc.has_bias ? dir + l1.b_off : nullptr;
    e.alpha = scale;
    e.e = h->f(h->fd_z1); e.Rz = eps; e.ldf = l1.n_out_p;
    e.dphi_out = h->f(sb.dphi[1]); e.d2_out = h->f(mb.dphi[1]);
    e.out = h->at<void>(sb.A[1]); e.outT = h->at<void>(sb.At[1]); e.out2 = h->at<void>(mb.A[1]); e.outT2 = h->at<void>(mb.At[1]);
    e.ld = l1.n_out_p; e.ldT = sb.Bp;
    chain_gemm(h, ELEM_F32, h->at<void>(sb.X), l1.n_in_p, h->at<void>(os.Wt[0]), l1.n_in_p, l1.n_in, nullptr, 0, nullptr, 0, 0,
               sb.B, l1.n_out, e, 2.0 * sb.B * l1.n_in * l1.n_out);
  };
  Pass ps[2] = {Pass{&os, 0, h->f(h->bias_pm[0])}, Pass{&om, 0, h->f(h->bias_pm[1])}};
  for (Pass& q : ps) q.omega_fixed = omega_bar;
  ps[1].sign = -1.f;
  auto both = [&](const float* dir, float scale, auto passes) {
    // Up to 4096 partial sums (32 KB, at most eight rounds of loads a thread beside those of the tile) every block of
    // the perturbation adds them up itself; beyond that a launch of one block forms the step: with
    // 5.3M parameters and 5 differences both take the same time (1282 and 1281 us).  Reweighting step 1023-509-251-10 with one difference: 145.3 -> 143.7 us.
    const int in_block = sums <= 4096 ? sums : 0;
    if (!in_block) launch_fd_eps(h->ctx, h->at<double>(h->sums), sums, eps_scale, scale, eps);
    for (int s = 0; s < (h->fd_paired ? 1 : 2); ++s) {
      make_perturbed_operands(h, w, dir, eps, scale, h->fd_paired ? 3 : 1 << s, in_block, eps_scale, !split);
      if (split && s == 0) first_layer(dir, scale);
      h->as_pair = true;
      h->layer1_done = split;
      passes(ps + s, h->fd_paired ? 2 : 1);
      h->as_pair = h->layer1_done = false;
    }
  };
  for (int k = 0; k < K; ++k) {
    both(v, 1.f, [&](const Pass* q, int n) { forward_backward(h, q, n); });
    const bool last = k + 1 == K;
    WgradSink step{last && !rw ? EPI_WGRAD_FD_LAST : EPI_WGRAD_FD, dlambda, dl, last && l2 ? w : nullptr, v, p, alpha, false};
    step.eps = eps;
    step.minus = &om;
    // Both points' gradients of layer 1 have the same left operand, so their deltas may be added (with their opposite
    // signs: the difference) before the product instead of after it.  A launch of 4 us against half of that product, at
    // some 70 TFLOP/s: from 2^28 multiplications.
    step.minus_summed = h->L >= 2 && products >= 268435456.0;
    step.sum_p = last;
    sums = 0;
    if (!last || rw) step.sums = &sums;
    if (step.minus_summed) {
      AccumulateBatch acc;
      acc.first = false; acc.last = true;
      acc.n = 1;
      acc.j[0] = AccumulateJob{h->at<void>(om.side[0].Dt[1]), h->f(sb.Dt[1]), 1.f, (size_t)l1.n_out_p * sb.Bp};
      launch_accumulate(h->ctx, ELEM_F32, acc);
    }
    wgrad_batch(h, os, 0, false, step);
  }
  const float* s = K > 0 ? p : v;
  if (rw) {
    // grad_theta L_L(w') = (1/B) sum_i l_i(w') dR(lbar_i)/dtheta, so its central difference along
    // q = alpha s needs only the per-sample losses at w +- eps q
    both(s, alpha, [&](const Pass* q, int n) { forward_and_loss(h, q, n); });
    launch_wnet_theta_vjp(h->ctx, h->f(sb.ell_bar), h->f(sb.dsig_bar), h->f(sb.ell), h->f(om.side[0].ell), eps, lambda,
                          h->desc.wnet_hidden, sb.B, 1.0f / (float)sb.B, dlambda);
  } else if (K == 0) {
    if (l2) launch_mixed_l2(h->ctx, lambda, w, s, alpha, dlambda, h->d, true);
    else launch_mixed_prox(h->ctx, h->f(h->logrho), s, alpha, dlambda, h->d);
  }
}

betty_status betty_hypergrad_fd(betty_handle h, const float* w, const float* lambda, int K, float alpha,
                                float eps_scale, float* dlambda) {
  CHECK(check_hyper_args(h, w, lambda, K, alpha, dlambda));
  if (!std::isfinite(eps_scale) || eps_scale <= 0.f) return fail(h, BETTY_EINVAL, "eps_scale must be positive and finite");
  auto body = [=]() { fd_seq(h, w, lambda, K, alpha, eps_scale, dlambda); };
  return run_cached(h, h->CALL_FD, call_key({w, lambda, dlambda}, K, {alpha, eps_scale}), body);
}

betty_status betty_hypergrad_cg(betty_handle h, const float* w, const float* lambda, int K, float* dlambda) {
  CHECK(check_hyper_args(h, w, lambda, K, 0.f, dlambda));
  if (use_linear(h, true, K)) { linear_seq(h, w, lambda, K, 0.f, dlambda, true); return finish(h); }
  auto body = [=]() {
    OperandSet& os = h->sets[0];
    const bool l2 = h->desc.hp == BETTY_HP_L2_DECAY, rw = h->desc.hp == BETTY_HP_REWEIGHT_NET;
    const float* dl = diag_log(h, lambda);
    float* r = h->f(h->vec_g); float* d = h->f(h->vec_v); float* q = h->f(h->vec_p); float* Hd = h->f(h->vec_Hv);
    float* sc = h->f(h->scalars);            // sc[0], sc[1]: r.r of the current / next iterate
    double* partials = h->at<double>(h->partials);
    make_weight_operands(h, os, w);
    int n_rs = 0;
    WgradSink init{EPI_WGRAD_INIT, nullptr, nullptr, nullptr, r, d, 0.f, K > 0};
    if (K > 0) init.sums = &n_rs;
    upper_grad_seq(h, os, w, lambda, K > 0 || rw, init, nullptr);
    if (K == 0) launch_fill_value(h->ctx, q, 0.f, h->d);
    for (int k = 0; k < K; ++k) {
      float* rs = sc + (k & 1);
      float* rs_new = sc + ((k + 1) & 1);
      const bool first = k == 0, last = k + 1 == K;
      int n_sums = (n_rs + 3) & ~3;
      const int begin = n_sums;
      WgradSink hd{EPI_WGRAD_CG, Hd, dl, d, nullptr, nullptr, 0.f, false};
      hd.sums = &n_sums;
      hvp_cached(h, os, d, hd);
      if (h->vec_r && !last) {
        CgUpdate u;
        u.n = h->L;
        u.q = q; u.r = r; u.r_out = r == h->f(h->vec_g) ? h->f(h->vec_r) : h->f(h->vec_g); u.d = d; u.Hd = Hd; u.params = (int)h->d;
        u.dHd = h->at<double>(h->sums) + begin; u.n_dHd = n_sums - begin;
        u.rs_partial = first ? h->at<double>(h->sums) : nullptr; u.n_rs = n_rs; u.rs = rs; u.rs_new = rs_new;
        for (int i = 0; i < h->L; ++i) {
          const LayerInfo& li = h->layers[i];
          u.j[i] = CgUpdateJob{(long long)li.w_off, h->desc.has_bias ? (long long)li.b_off : -1LL, li.n_in, li.n_out,
                               i > 0 ? h->at<void>(os.Vn[i]) : nullptr, li.n_out_p, h->at<void>(os.Vt[i]), li.n_in_p};
        }
        launch_cg_update(h->ctx, os.elem, u);
        r = u.r_out;
        continue;
      }
      CgStep c{q, r, d, Hd, h->d, h->at<double>(h->sums) + begin, n_sums - begin, first ? h->at<double>(h->sums) : nullptr, n_rs, rs, partials};
      if (last && !rw) { c.lam = dl; c.w = l2 ? w : nullptr; c.out = dlambda; }
      const int n_partial = launch_cg_step(h->ctx, c);
      if (last) break;
      for (int i0 = 0; i0 < h->L; i0 += MAX_PROBLEMS) {
        CgDirBatch b;
        b.n = std::min(MAX_PROBLEMS, h->L - i0);
        b.partials = partials; b.n_partial = n_partial; b.rs = rs; b.rs_new = i0 == 0 ? rs_new : nullptr;
        for (int i = 0; i < b.n; ++i) {
          const LayerInfo& li = h->layers[i0 + i];
          b.j[i] = CgDirJob{r + li.w_off, d + li.w_off, li.n_in, li.n_out,
                             i0 + i > 0 ? h->at<void>(os.Vn[i0 + i]) : nullptr, li.n_out_p,
                            h->at<void>(os.Vt[i0 + i]), li.n_in_p, h->desc.has_bias ? r + li.b_off : nullptr,
                            h->desc.has_bias ? d + li.b_off : nullptr};
        }
        launch_cg_dir(h->ctx, os.elem, b);
      }
    }
    if (K > 0 && !rw) return;
    if (l2) launch_mixed_l2(h->ctx, lambda, w, q, 1.f, dlambda, h->d);
    else if (rw) mixed_reweight_seq(h, os, lambda, q, 1.f, dlambda);
    else launch_mixed_prox(h->ctx, h->f(h->logrho), q, 1.f, dlambda, h->d);
  };
  return run_cached(h, h->CALL_CG, call_key({w, lambda, dlambda}, K), body);
}

betty_status betty_lower_sgd_step(betty_handle h, float* w, const float* lambda, float* momentum, float lr, float mu,
                                  float weight_decay, float* loss_or_null) {
  CHECK(check_ready(h));
  CHECK(check_vec(h, w, "w")); CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, momentum, "momentum"));
  if (loss_or_null) CHECK(check_vec(h, loss_or_null, "loss"));
  if (!std::isfinite(lr) || !std::isfinite(mu) || !std::isfinite(weight_decay))
    return fail(h, BETTY_EINVAL, "lr, mu and weight_decay must be finite");
  if (overlaps(w, h->d * 4, momentum, h->d * 4) || overlaps(w, h->d * 4, lambda, h->n_hyper * 4) ||
      overlaps(momentum, h->d * 4, lambda, h->n_hyper * 4))
    return fail(h, BETTY_EINVAL, "w, momentum and lambda must not overlap");
  return run_cached(h, h->CALL_SGD, call_key({w, lambda, momentum, loss_or_null}, -1, {lr, mu, weight_decay}), [=]() {
    OperandSet& os = h->sets[0];
    const bool prox = h->desc.hp == BETTY_HP_PROXIMAL;
    const float* dl = diag_log(h, lambda);
    make_weight_operands(h, os, w);
    const Pass ps = train_pass(h, os, w, lambda, false);
    h->fixed_grouping = true;
    forward_backward(h, &ps, 1);
    h->fixed_grouping = false;
    // momentum and parameters are updated in the epilogue of the weight-gradient launch
    // (the proximal term pulls towards the anchor: the epilogue subtracts it from w in that term)
    WgradSink k{EPI_WGRAD_SGD, nullptr, dl, prox ? lambda : nullptr, momentum, w, lr, false};
    k.beta = mu; k.gamma = weight_decay;
    int n = 0;
    if (dl && loss_or_null) k.sums = &n;
    wgrad_batch(h, os, 0, false, k);
    if (loss_or_null)                        // the cost at the w before the step
      launch_weighted_loss_sum(h->ctx, h->f(os.side[0].s), h->f(os.side[0].ell), os.side[0].B, h->at<double>(h->sums), n, loss_or_null);
  });
}

betty_status betty_upper_adam_step(betty_handle h, float* lambda, const float* dlambda, float* m, float* v, int t,
                                   float lr, float beta1, float beta2, float eps) {
  if (!h) return BETTY_ENULL;
  CHECK(check_vec(h, lambda, "lambda")); CHECK(check_vec(h, dlambda, "dlambda")); CHECK(check_vec(h, m, "m"));
  CHECK(check_vec(h, v, "v"));
  if (t < 1) return fail(h, BETTY_EINVAL, "t must be >= 1 (got %d)", t);
  if (!std::isfinite(lr) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f))
    return fail(h, BETTY_EINVAL, "need finite lr, 0 <= beta1, beta2 < 1, eps >= 0");
  const size_t nb = h->n_hyper * 4;
  if (overlaps(lambda, nb, dlambda, nb) || overlaps(lambda, nb, m, nb) || overlaps(lambda, nb, v, nb) ||
      overlaps(m, nb, v, nb) || overlaps(m, nb, dlambda, nb) || overlaps(v, nb, dlambda, nb))
    return fail(h, BETTY_EINVAL, "lambda, dlambda, m and v must not overlap");
  const float bias1 = 1.f - std::pow(beta1, (float)t), bias2 = 1.f - std::pow(beta2, (float)t);
  launch_adam(h->ctx, lambda, dlambda, m, v, lr, beta1, beta2, eps, bias1, bias2, h->n_hyper);
  return finish(h);
}

betty_status betty_apply_label_noise(betty_handle h, const int32_t* y, const uint32_t* words, const int32_t* alt,
                                     double p, int n, int32_t* y_out, uint8_t* mask_or_null) {
  if (!h) return BETTY_ENULL;
  if (n < 0) return fail(h, BETTY_EINVAL, "n must be >= 0");
  if (!(p >= 0.0 && p <= 1.0)) return fail(h, BETTY_EINVAL, "p must lie in [0, 1]");
  if (n == 0) return BETTY_OK;
  CHECK(check_vec(h, y, "y")); CHECK(check_vec(h, words, "words")); CHECK(check_vec(h, alt, "alt"));
  CHECK(check_vec(h, y_out, "y_out"));
  unsigned long long T = (unsigned long long)std::floor(p * 4294967296.0);
  if (T > 4294967296ULL) T = 4294967296ULL;
  launch_label_noise(h->ctx, y, words, alt, T, n, y_out, mask_or_null);
  return finish(h);
}

betty_status betty_profile_enable(betty_handle h, int on) {
  if (!h) return BETTY_ENULL;
  for (auto& r : h->ctx.recs) { (void)hipEventDestroy(r.e0); (void)hipEventDestroy(r.e1); }
  h->ctx.recs.clear();
  h->ctx.profiling = on != 0;
  return BETTY_OK;
}

int betty_profile_collect(betty_handle h) {
  if (!h) return 0;
  if (hipStreamSynchronize(h->ctx.stream) != hipSuccess) return 0;
  for (auto& r : h->ctx.recs)
    if (r.ms < 0.f && hipEventElapsedTime(&r.ms, r.e0, r.e1) != hipSuccess) r.ms = -1.f;
  return (int)h->ctx.recs.size();
}

betty_status betty_profile_get(betty_handle h, int i, betty_profile_rec* out) {
  if (!h || !out) return BETTY_ENULL;
  if (i < 0 || i >= (int)h->ctx.recs.size()) return fail(h, BETTY_EINVAL, "profile record %d out of range", i);
  const ProfRec& r = h->ctx.recs[i];
  out->kind = r.kind; out->ms = r.ms; out->flops = r.flops; out->bytes = r.bytes;
  return BETTY_OK;
}

}  // extern "C"
