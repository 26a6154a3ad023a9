// Composition of one GNN layer, forward and backward, from the aggregation and dense kernels
// (layer definition of Section 3; gradient flow as in the proof of Theorem 3).
#include <cstdint>
#include <cstdlib>
#include <mutex>

#include "common.h"

namespace cofree {

// ---- a second stream for work that does not depend on the aggregation chain -------------------
// In backward the weight gradients that only need the incoming gradient (compute bound) are
// independent of the transposed aggregation (memory bound); with COFREE_OVERLAP=1 in the environment
// they are enqueued on a library-owned stream between a fork event (recorded on the caller's stream)
// and a join event (waited on by the caller's stream before the call returns control of the
// outputs), so the two overlap.  Default priority, created once per device.  Off by default: both
// kernels are bound inside the compute unit and mostly take turns on it, so the step gains 0-3 %
// while every kernel's own duration, as events see it, grows by up to half.
struct SideStream {
  hipStream_t stream = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  bool ok = false;
};

static SideStream* side_stream() {
  static std::mutex mu;
  static SideStream per_device[64];
  static bool tried[64];
  const char* env = getenv("COFREE_OVERLAP");
  if (!env || atoi(env) == 0) return nullptr;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(mu);
  SideStream& s = per_device[dev];
  if (!tried[dev]) {
    tried[dev] = true;
    s.ok = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) == hipSuccess &&
           hipEventCreateWithFlags(&s.fork, hipEventDisableTiming) == hipSuccess &&
           hipEventCreateWithFlags(&s.join, hipEventDisableTiming) == hipSuccess;
  }
  return s.ok ? &s : nullptr;
}

// Returns the stream to use for the independent work: the side stream (after it has been made to
// wait for everything enqueued on `main` so far), or `main` itself if overlap is unavailable.
static hipStream_t fork_side(hipStream_t main, SideStream** used) {
  *used = nullptr;
  SideStream* s = side_stream();
  if (!s) return main;
  if (hipEventRecord(s->fork, main) != hipSuccess) return main;
  if (hipStreamWaitEvent(s->stream, s->fork, 0) != hipSuccess) return main;
  *used = s;
  return s->stream;
}

static int32_t join_side(hipStream_t main, SideStream* s) {
  if (!s) return COFREE_OK;
  COFREE_HIP_CHECK(hipEventRecord(s->join, s->stream));
  COFREE_HIP_CHECK(hipStreamWaitEvent(main, s->join, 0));
  return COFREE_OK;
}

// Joins the side stream back into the caller's stream when the call leaves, also on an error path.
struct SideJoin {
  hipStream_t main;
  SideStream* side;
  ~SideJoin() { (void)join_side(main, side); }
  int32_t finish() {
    SideStream* s = side;
    side = nullptr;
    return join_side(main, s);
  }
};

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static inline size_t elem_size(int32_t dtype) { return dtype == COFREE_BF16 ? 2 : 4; }

// Carves 256-byte aligned buffers out of the caller's workspace.
struct Carver {
  char* base;
  size_t used = 0;
  explicit Carver(void* p) : base((char*)p) {}
  void* take(size_t bytes) {
    void* r = base ? (void*)(base + used) : nullptr;
    used += align256(bytes);
    return r;
  }
};

static bool gcn_transform_first(const cofree_layer_desc& d) { return d.d_out < d.d_in; }
// Conventional GraphSAGE: the mean commutes with W_neigh, so it runs on min(d_in, d_out) columns.
static bool conv_transform_first(const cofree_layer_desc& d) { return d.d_out < d.d_in; }
// In backward the transposed mean runs on the columns of the outgoing gradient up to equal widths: mean^T(dPre) and one
// product over [dPre | mean^T(dPre)] move 5 matrices of n x d, mean^T(dPre W_neigh) with dPre W_self added to it 7, and
// one rounding of the storage type falls away.  Measured: 1.88M x 128 bfloat16 0.91 -> 0.72 ms, 529k x 512 float32
// 3.61 -> 3.31 (two products of 512 k against one of 1024).
static bool conv_gathers_grad(const cofree_layer_desc& d) { return d.d_out <= d.d_in; }
// The neighbourhood mean commutes with the linear map U_a, so when the layer output is narrower
// than the messages the mean is taken after U_a (on d_out columns instead of d_msg).
static bool sage_combine_first(const cofree_layer_desc& d) { return d.d_out < d.d_msg; }

// Two weight gradients of a layer that share the incoming gradient are one launch when both blocks are whole numbers of
// 128-column tiles, or in bfloat16 when they fit one tile: the incoming gradient is read once (the products are memory
// bound in bf16; 256x512 over 1.9M nodes 0.72 ms against 2 x 0.40; with a ragged second block in a tile of its own the
// merged launch measured slower; 128x(100+100) 379 -> 243 us).
static bool merged_widths(const cofree_layer_desc& d, int32_t first, int32_t second) {
  if (first % 128 == 0 && second % 128 == 0) return true;
  return d.dtype == COFREE_BF16 && wgrad_bf16_fits(d.d_out, first, second) && (first + 7) / 8 + (second + 7) / 8 <= 32;
}
static bool sage_merged(const cofree_layer_desc& d) {
  return !sage_combine_first(d) && merged_widths(d, d.d_msg, d.d_in);
}
static bool conv_merged(const cofree_layer_desc& d) {
  return d.kind == COFREE_SAGE_CONV && !conv_transform_first(d) && merged_widths(d, d.d_in, d.d_in);
}

static size_t max2(size_t a, size_t b) { return a > b ? a : b; }
static size_t max3(size_t a, size_t b, size_t c) { return max2(a, max2(b, c)); }

// Conventional GraphSAGE, transform first: both products of H are one launch, and the self part is added by the
// aggregation - H is read once, and a launch falls away.
static bool conv_two(const cofree_layer_desc& d, int64_t n) {
  return d.kind == COFREE_SAGE_CONV && d.dtype == COFREE_F32 && conv_transform_first(d) && gemm_two_fits(d.d_out, d.d_in, n);
}

// largest copy of a parameter matrix - in bfloat16, or split into three of them - that any product of the layer makes.  In
// float32 it only saves time: a call whose workspace has no room for it does without.
static size_t param_scratch_bytes(const cofree_layer_desc& d, int64_t n) {
  if (d.dtype != COFREE_BF16) {
    if (d.kind == COFREE_SAGE_MEAN)
      return max3(split_param_bytes(n, d.d_msg, d.d_in, 0), split_param_bytes(n, d.d_out, d.d_msg, d.d_in),
                  max2(split_param_bytes(n, d.d_msg, d.d_out, 0), split_param_bytes(n, d.d_in, d.d_out, d.d_msg)));
    if (d.kind == COFREE_SAGE_CONV)
      return max3(split_param_bytes(n, d.d_out, d.d_in, d.d_in), split_param_bytes(n, d.d_in, d.d_out, d.d_out),
                  conv_two(d, n) ? split_param_bytes(n, 2 * d.d_out, d.d_in, 0) : 0);
    return max2(split_param_bytes(n, d.d_out, d.d_in, 0), split_param_bytes(n, d.d_in, d.d_out, 0));
  }
  if (d.kind == COFREE_SAGE_MEAN)
    return max3(gemm_param_scratch_bytes(d.d_msg, d.d_in),
                gemm_param_scratch_bytes(d.d_out, (int64_t)d.d_msg + d.d_in),
                max2(gemm_param_scratch_bytes(d.d_msg, d.d_out),
                     gemm_param_scratch_bytes(d.d_in, (int64_t)d.d_out + d.d_msg)));
  if (d.kind == COFREE_SAGE_CONV)
    return max2(gemm_param_scratch_bytes(d.d_out, 2 * (int64_t)d.d_in),
                gemm_param_scratch_bytes(d.d_in, 2 * (int64_t)d.d_out));
  return max2(gemm_param_scratch_bytes(d.d_out, d.d_in), gemm_param_scratch_bytes(d.d_in, d.d_out));
}

// ... and both weight gradients, of dPre and mean^T(dPre), which read H too.
static bool conv_two_wgrads(const cofree_layer_desc& d, int64_t n) {
  return d.kind == COFREE_SAGE_CONV && conv_transform_first(d) && wgrad_two_fits(d.dtype, d.d_out, d.d_in, n);
}

struct FwdPlan {
  void* T = nullptr;       // transform-first: norm * (H W^T) (GCN), H W_neigh^T (conventional GraphSAGE)
  void* S = nullptr;       // H W_self^T where both products are one launch
  void* params = nullptr;  // copy of a parameter matrix
  size_t params_bytes = 0;
  size_t bytes = 0, needed = 0;  // in all; of which a call cannot do without
};

// room: bytes of the workspace (two results only where they find room)
static FwdPlan plan_fwd(const cofree_layer_desc& d, int64_t n, void* ws, size_t room) {
  Carver c(ws);
  FwdPlan p;
  const size_t T = (size_t)n * d.d_out * elem_size(d.dtype);
  if ((d.kind == COFREE_GCN && gcn_transform_first(d)) || (d.kind == COFREE_SAGE_CONV && conv_transform_first(d))) p.T = c.take(T);
  if (conv_two(d, n) && room >= c.used + align256(T)) p.S = c.take(T);
  p.needed = c.used;
  p.params_bytes = param_scratch_bytes(d, n);
  p.params = c.take(p.params_bytes);
  p.bytes = c.used;
  if (d.dtype == COFREE_BF16) p.needed = p.bytes;
  return p;
}

struct BwdPlan {
  void *dP = nullptr, *dA = nullptr, *dZ = nullptr, *T = nullptr, *params = nullptr;
  // partials of up to three weight gradients (they stay until they are summed), one behind the other, of one bias gradient
  float *wg[3] = {nullptr, nullptr, nullptr}, *cs = nullptr;
  size_t params_bytes = 0;
  size_t needed = 0;  // bytes of the layer's own workspace that a call cannot do without
};

// c: what is dead when the layer is done; part: the partials (the same carver where a layer sums its own)
static BwdPlan plan_bwd(const cofree_layer_desc& d, int64_t n, Carver& c, Carver& part) {
  BwdPlan p;
  const size_t N = (size_t)n, es = elem_size(d.dtype);
  if (d.kind == COFREE_SAGE_MEAN) {
    if (d.dropout_q > 0.f) p.dP = c.take(N * d.d_out * es);
    p.dA = c.take(N * d.d_msg * es);
    p.dZ = c.take(N * d.d_msg * es);
    if (sage_merged(d)) {
      p.wg[0] = (float*)part.take(4 * wgrad_workspace_floats(d.d_out, d.d_msg, n, d.d_in));
    } else {
      p.wg[0] = (float*)part.take(4 * wgrad_workspace_floats(d.d_out, d.d_in, n));
      p.wg[1] = (float*)part.take(4 * wgrad_workspace_floats(d.d_out, d.d_msg, n));
    }
    p.wg[2] = (float*)part.take(4 * wgrad_workspace_floats(d.d_msg, d.d_in, n));
  } else {
    if (d.dropout_q > 0.f || d.act) p.dP = c.take(N * d.d_out * es);
    // transform first: T = Ahat dPre [n, d_out]; aggregate first: T = norm * (dPre W) [n, d_in]
    p.T = c.take(N * (gcn_transform_first(d) ? d.d_out : d.d_in) * es);
    p.wg[0] = (float*)part.take(4 * wgrad_workspace_floats(d.d_out, d.d_in, n, conv_merged(d) ? d.d_in : 0));
    if (d.kind == COFREE_SAGE_CONV && !conv_merged(d)) p.wg[1] = (float*)part.take(4 * wgrad_workspace_floats(d.d_out, d.d_in, n));
    if (d.kind == COFREE_GCN && gcn_transform_first(d)) p.cs = (float*)part.take(4 * colsum_workspace_floats(d.d_out));
  }
  p.needed = c.used;
  p.params_bytes = param_scratch_bytes(d, n);
  p.params = c.take(p.params_bytes);
  if (d.dtype == COFREE_BF16) p.needed = c.used;
  return p;
}

static size_t bwd_bytes(const cofree_layer_desc& d, int64_t n) {
  Carver c(nullptr);
  plan_bwd(d, n, c, c);
  return c.used;
}

// The layers of a backward pass may leave their partials until one launch sums all of them: a launch less per layer, which
// is what small graphs wait for (2,000 nodes, two layers 69.4 -> 66.5 us a training step).  Beyond DEFER_MAX bytes of partials the sums of a layer take
// longer than a launch does, and every layer uses the same part of the workspace.
constexpr size_t DEFER_MAX = (size_t)32 << 20;
struct Deferral {
  size_t scratch = 0, partials = 0;  // bytes: shared by the layers in turn; of all layers
  bool worth = false;
};
template <typename Desc>
static Deferral plan_deferral(int32_t n_layers, int64_t n, const Desc& desc) {
  Deferral f;
  for (int32_t l = 0; l < n_layers; ++l) {
    Carver c(nullptr), part(nullptr);
    plan_bwd(desc(l), n, c, part);
    f.scratch = max2(f.scratch, c.used);
    f.partials += part.used;
  }
  f.worth = n_layers > 1 && f.partials <= DEFER_MAX;
  return f;
}

static int32_t check_desc(const cofree_layer_desc* d) {
  COFREE_REQUIRE(d != nullptr, "layer: desc is NULL");
  COFREE_REQUIRE(d->kind == COFREE_GCN || d->kind == COFREE_SAGE_MEAN || d->kind == COFREE_SAGE_CONV,
                 "layer: unknown kind");
  COFREE_REQUIRE(d->dtype == COFREE_F32 || d->dtype == COFREE_BF16, "layer: unknown dtype");
  COFREE_REQUIRE(d->d_in >= 1 && d->d_out >= 1, "layer: d_in and d_out must be >= 1");
  COFREE_REQUIRE(d->kind != COFREE_SAGE_MEAN || d->d_msg >= 1, "layer: d_msg must be >= 1");
  COFREE_REQUIRE(d->dropout_q >= 0.f && d->dropout_q < 1.f, "layer: dropout_q must be in [0, 1)");
  COFREE_REQUIRE(d->layer_id >= 0 && d->layer_id < (1 << 23), "layer: layer_id out of range");
  COFREE_REQUIRE((d->grad_flags & ~(COFREE_GRAD_IN_GATED | COFREE_GRAD_OUT_GATED)) == 0, "layer: unknown grad_flags");
  COFREE_REQUIRE(d->dropout_q_below >= 0.f && d->dropout_q_below < 1.f, "layer: dropout_q_below must be in [0, 1)");
  COFREE_REQUIRE(!(d->grad_flags & COFREE_GRAD_IN_GATED) || d->kind != COFREE_SAGE_MEAN,
                 "layer: COFREE_GRAD_IN_GATED is for GCN and SAGE_CONV layers");
  COFREE_REQUIRE(!(d->grad_flags & COFREE_GRAD_OUT_GATED) || (d->kind != COFREE_SAGE_MEAN && d->act),
                 "layer: COFREE_GRAD_OUT_GATED needs a layer that ends in ReLU");
  return COFREE_OK;
}

static DropoutArgs dropout_of(const cofree_layer_desc& d) {
  DropoutArgs o;
  o.q = d.dropout_q;
  o.seed = d.seed;
  o.epoch = (uint32_t)d.epoch;
  o.layer_id = (uint32_t)d.layer_id;
  return o;
}

}  // namespace cofree

using namespace cofree;

extern "C" {

size_t cofree_layer_desc_size(void) { return sizeof(cofree_layer_desc); }

size_t cofree_layer_workspace_bytes(const cofree_layer_desc* desc, int64_t n_nodes, int32_t backward) {
  if (!desc || n_nodes < 0) return 0;
  const size_t b = backward ? bwd_bytes(*desc, n_nodes) : plan_fwd(*desc, n_nodes, nullptr, SIZE_MAX).bytes;
  return b < 256 ? 256 : b;
}

int32_t cofree_layer_fwd(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                         const cofree_layer_desc* desc, const void* H_in, const cofree_layer_params* params,
                         void* H_out, const cofree_layer_saved* saved, void* workspace, size_t workspace_bytes,
                         void* stream) {
  COFREE_TRY(check_desc(desc));
  const cofree_layer_desc& d = *desc;
  DeviceGraph g;
  COFREE_TRY(select_graph(part, masks, mask_id, &g));
  COFREE_REQUIRE(H_in && H_out && params && saved, "layer_fwd: NULL argument");
  COFREE_REQUIRE(params->W && params->bW, "layer_fwd: W / bW is NULL");
  const FwdPlan fp = plan_fwd(d, g.n, workspace, workspace ? workspace_bytes : 0);
  if (fp.needed > 0 && (workspace == nullptr || workspace_bytes < fp.needed))
    return fail(COFREE_ENOMEM, "layer_fwd: workspace too small");
  const bool copies = workspace != nullptr && workspace_bytes >= fp.bytes;
  hipStream_t s = (hipStream_t)stream;
  const int64_t n = g.n;
  const int32_t dt = d.dtype;
  auto gemm = [&]() {
    GemmArgs a;
    a.dtype = dt;
    if (copies) a.param_scratch = fp.params, a.param_scratch_bytes = fp.params_bytes;
    a.M = n;
    return a;
  };
  auto agg = [&]() {
    AggArgs a;
    a.g = g;
    a.dtype = dt;
    return a;
  };

  // Inverted dropout of the layer's output (the same keep decisions are recomputed in backward) is applied by the launch
  // that finishes H_out where its kernel can, else in place by a launch of its own (which wants H_out aligned)
  bool dropped = false;
  auto with_dropout = [&](auto& last, bool can) {
    if (d.dropout_q > 0.f && can && ((uintptr_t)H_out & 15u) == 0) {
      last.dropout = dropout_of(d);
      dropped = true;
    }
  };

  if (d.kind == COFREE_SAGE_MEAN) {
    COFREE_REQUIRE(params->U && params->bU, "layer_fwd: U / bU is NULL");
    COFREE_REQUIRE(saved->Z && saved->A, "layer_fwd: saved.Z / saved.A is NULL");
    void* Z = saved->Z;
    void* A = saved->A;
    const int64_t ldu = (int64_t)d.d_msg + d.d_in;
    // messages: Z = ReLU(H W^T + bW)
    GemmArgs m = gemm();
    m.A1 = H_in; m.lda1 = d.d_in; m.K1 = d.d_in;
    m.B = params->W; m.ldb = d.d_in;
    m.C = Z; m.ldc = d.d_msg; m.N = d.d_msg;
    m.bias = params->bW; m.relu = 1;
    COFREE_TRY(launch_gemm(m, s));
    if (sage_combine_first(d)) {
      // H' = mean(Z U_a^T) + H U_s^T + bU: T = Z U_a^T is kept in the A buffer
      GemmArgs t = gemm();
      t.A1 = Z; t.lda1 = d.d_msg; t.K1 = d.d_msg;
      t.B = params->U; t.ldb = ldu;
      t.C = A; t.ldc = d.d_out; t.N = d.d_out;
      COFREE_TRY(launch_gemm(t, s));
      AggArgs a = agg();
      a.X = A; a.Y = H_out; a.width = d.d_out; a.ldx = a.ldy = d.d_out;
      a.out_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(a, s));
      GemmArgs c = gemm();
      c.A1 = H_in; c.lda1 = d.d_in; c.K1 = d.d_in;
      c.B = params->U + d.d_msg; c.ldb = ldu;
      c.C = H_out; c.ldc = d.d_out; c.N = d.d_out;
      c.bias = params->bU; c.accumulate = 1;
      with_dropout(c, gemm_drops(c));
      COFREE_TRY(launch_gemm(c, s));
    } else {
      // neighbourhood mean, then combine: H' = [A | H] U^T + bU
      AggArgs a = agg();
      a.X = Z; a.Y = A; a.width = d.d_msg; a.ldx = a.ldy = d.d_msg;
      a.out_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(a, s));
      GemmArgs c = gemm();
      c.A1 = A; c.lda1 = d.d_msg; c.K1 = d.d_msg;
      c.A2 = H_in; c.lda2 = d.d_in; c.K2 = d.d_in;
      c.B = params->U; c.ldb = ldu;
      c.C = H_out; c.ldc = d.d_out; c.N = d.d_out;
      c.bias = params->bU;
      with_dropout(c, gemm_drops(c));
      COFREE_TRY(launch_gemm(c, s));
    }
  } else if (d.kind == COFREE_SAGE_CONV) {
    const int64_t ldw = 2 * (int64_t)d.d_in;  // W = [W_self | W_neigh]
    if (fp.S) {
      // T = H W_neigh^T, S = H W_self^T; H' = act(mean(T) + (S + b))
      GemmArgs t = gemm();
      t.A1 = H_in; t.lda1 = d.d_in; t.K1 = d.d_in;
      t.B = params->W + d.d_in; t.ldb = ldw;
      t.C = fp.T; t.ldc = d.d_out; t.N = d.d_out;
      t.B_second = params->W; t.C_second = fp.S;
      COFREE_TRY(launch_gemm(t, s));
      AggArgs a = agg();
      a.X = fp.T; a.Y = H_out; a.width = d.d_out; a.ldx = a.ldy = d.d_out;
      a.out_scale = g.inv_deg;
      a.add = fp.S; a.ld_add = d.d_out;
      a.bias = params->bW; a.relu_out = d.act;
      with_dropout(a, aggregate_drops(a));
      COFREE_TRY(launch_aggregate(a, s));
    } else if (conv_transform_first(d)) {
      // T = H W_neigh^T; H' = mean(T); H' = act(H' + H W_self^T + b)
      GemmArgs t = gemm();
      t.A1 = H_in; t.lda1 = d.d_in; t.K1 = d.d_in;
      t.B = params->W + d.d_in; t.ldb = ldw;
      t.C = fp.T; t.ldc = d.d_out; t.N = d.d_out;
      COFREE_TRY(launch_gemm(t, s));
      AggArgs a = agg();
      a.X = fp.T; a.Y = H_out; a.width = d.d_out; a.ldx = a.ldy = d.d_out;
      a.out_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(a, s));
      GemmArgs c = gemm();
      c.A1 = H_in; c.lda1 = d.d_in; c.K1 = d.d_in;
      c.B = params->W; c.ldb = ldw;
      c.C = H_out; c.ldc = d.d_out; c.N = d.d_out;
      c.bias = params->bW; c.accumulate = 1; c.relu_last = d.act;
      with_dropout(c, gemm_drops(c));
      COFREE_TRY(launch_gemm(c, s));
    } else {
      COFREE_REQUIRE(saved->A, "layer_fwd: saved.A is NULL");
      // M = mean(H), then H' = act([H | M] W^T + b)
      AggArgs a = agg();
      a.X = H_in; a.Y = saved->A; a.width = d.d_in; a.ldx = a.ldy = d.d_in;
      a.out_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(a, s));
      GemmArgs c = gemm();
      c.A1 = H_in; c.lda1 = d.d_in; c.K1 = d.d_in;
      c.A2 = saved->A; c.lda2 = d.d_in; c.K2 = d.d_in;
      c.B = params->W; c.ldb = ldw;
      c.C = H_out; c.ldc = d.d_out; c.N = d.d_out;
      c.bias = params->bW; c.relu = d.act;
      with_dropout(c, gemm_drops(c));
      COFREE_TRY(launch_gemm(c, s));
    }
  } else if (gcn_transform_first(d)) {
    // T = norm * (H W^T), then H' = act(norm * (T[v] + sum T[u]) + b)
    GemmArgs t = gemm();
    t.A1 = H_in; t.lda1 = d.d_in; t.K1 = d.d_in;
    t.B = params->W; t.ldb = d.d_in;
    t.C = fp.T; t.ldc = d.d_out; t.N = d.d_out;
    t.row_scale = g.gcn_norm;
    COFREE_TRY(launch_gemm(t, s));
    AggArgs a = agg();
    a.X = fp.T; a.Y = H_out; a.width = d.d_out; a.ldx = a.ldy = d.d_out;
    a.out_scale = g.gcn_norm; a.self_loop = 1;  // sources are already scaled
    a.bias = params->bW; a.relu_out = d.act;
    with_dropout(a, aggregate_drops(a));
    COFREE_TRY(launch_aggregate(a, s));
  } else {
    COFREE_REQUIRE(saved->A, "layer_fwd: saved.A is NULL");
    // P = Ahat H, then H' = act(P W^T + b)
    AggArgs a = agg();
    a.X = H_in; a.Y = saved->A; a.width = d.d_in; a.ldx = a.ldy = d.d_in;
    a.in_scale = g.gcn_norm; a.out_scale = g.gcn_norm; a.self_loop = 1;
    COFREE_TRY(launch_aggregate(a, s));
    GemmArgs t = gemm();
    t.A1 = saved->A; t.lda1 = d.d_in; t.K1 = d.d_in;
    t.B = params->W; t.ldb = d.d_in;
    t.C = H_out; t.ldc = d.d_out; t.N = d.d_out;
    t.bias = params->bW; t.relu = d.act;
    with_dropout(t, gemm_drops(t));
    COFREE_TRY(launch_gemm(t, s));
  }
  if (d.dropout_q > 0.f && !dropped) COFREE_TRY(launch_mask_grad(dt, H_out, nullptr, H_out, n, d.d_out, dropout_of(d), s));
  return COFREE_OK;
}

}  // extern "C"

// Launches the first `before` sums by themselves where one of the others goes to the same memory.
static int32_t sums_of_one_launch(SplitSums* sums, int32_t before, hipStream_t s) {
  auto last = [](const SplitSum& j) { return j.C + (int64_t)(j.rows - 1) * j.ldc + j.cols; };
  bool meet = false;
  for (int32_t a = 0; a < before; ++a)
    for (int32_t b = before; b < sums->n; ++b)
      meet = meet || (sums->job[a].C < last(sums->job[b]) && sums->job[b].C < last(sums->job[a]));
  if (!meet) return COFREE_OK;
  SplitSums first = *sums;
  first.n = before;
  COFREE_TRY(launch_split_sums(first, s));
  for (int32_t b = before; b < sums->n; ++b) sums->job[b - before] = sums->job[b];
  sums->n -= before;
  return COFREE_OK;
}

// One layer's backward pass, which leaves its weight and bias gradients as partials in `sums`.  partials: the part of the
// workspace that they go to, null where they follow the layer's scratch.
static int32_t layer_bwd(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                         const cofree_layer_desc* desc, const void* H_in, const void* H_out,
                         const cofree_layer_params* params, const cofree_layer_saved* saved, const void* dH_out,
                         void* dH_in, const cofree_layer_grads* grads, void* workspace, size_t workspace_bytes,
                         Carver* partials, SplitSums* sums, hipStream_t s) {
  COFREE_TRY(check_desc(desc));
  const cofree_layer_desc& d = *desc;
  DeviceGraph g;
  COFREE_TRY(select_graph(part, masks, mask_id, &g));
  COFREE_REQUIRE(H_in && H_out && params && saved && dH_out && grads && workspace, "layer_bwd: NULL argument");
  COFREE_REQUIRE(params->W && grads->W && grads->bW, "layer_bwd: W / grads.W / grads.bW is NULL");
  const int64_t n = g.n;
  Carver scratch(workspace);
  const BwdPlan p = plan_bwd(d, n, scratch, partials ? *partials : scratch);
  if (workspace_bytes < p.needed) return fail(COFREE_ENOMEM, "layer_bwd: workspace too small");
  const bool copies = workspace_bytes >= scratch.used;
  const int32_t dt = d.dtype;
  auto gemm = [&]() {
    GemmArgs a;
    a.dtype = dt;
    if (copies) a.param_scratch = p.params, a.param_scratch_bytes = p.params_bytes;
    a.M = n;
    return a;
  };
  auto agg = [&]() {
    AggArgs a;
    a.g = g;
    a.dtype = dt;
    return a;
  };
  auto wgrad = [&](const void* A, int32_t N1, const void* B, int32_t N2, float* C, int64_t ldc, float* ws) {
    WgradArgs a;
    a.dtype = dt;
    a.M = n;
    a.A = A; a.lda = N1; a.N1 = N1;
    a.B = B; a.ldb = N2; a.N2 = N2;
    a.C = C; a.ldc = ldc;
    a.workspace = ws;
    return a;
  };

  if (d.kind == COFREE_SAGE_MEAN) {
    COFREE_REQUIRE(params->U && grads->U && grads->bU, "layer_bwd: U / grads.U / grads.bU is NULL");
    COFREE_REQUIRE(saved->Z && saved->A, "layer_bwd: saved.Z / saved.A is NULL");
    const void* Z = saved->Z;
    const void* A = saved->A;
    const int64_t ldu = (int64_t)d.d_msg + d.d_in;
    // gradient at the combine output (undo dropout scaling)
    const void* dP = dH_out;
    if (d.dropout_q > 0.f) {
      COFREE_TRY(launch_mask_grad(dt, dH_out, nullptr, p.dP, n, d.d_out, dropout_of(d), s));
      dP = p.dP;
    }
    // dU_s = dP^T H and dbU = column sums of dP need only dP: side stream
    SideStream* side = nullptr;
    hipStream_t s2 = fork_side(s, &side);
    SideJoin joiner{s, side};
    // dU = dP^T [A | H], in one launch or two
    const bool merged_dU = sage_merged(d);
    WgradArgs u = merged_dU ? wgrad(dP, d.d_out, A, d.d_msg, grads->U, ldu, p.wg[0])
                            : wgrad(dP, d.d_out, H_in, d.d_in, grads->U + d.d_msg, ldu, p.wg[0]);
    if (merged_dU) u.B2 = H_in, u.ldb2 = u.N2b = d.d_in;
    u.colsum_out = grads->bU;
    if (sage_combine_first(d)) {
      const WgradArgs ua = wgrad(p.dA, d.d_out, Z, d.d_msg, grads->U, ldu, p.wg[1]);
      const bool together = !side && wgrads_pair(u, ua);  // one launch instead of two
      if (!together) COFREE_TRY(launch_wgrad(u, sums, s2));
      // forward was mean(Z U_a^T): dT = mean^T(dP) on d_out columns, dU_a = dT^T Z,
      // dZ = [Z > 0] * (dT U_a)
      AggArgs t = agg();
      t.X = dP; t.Y = p.dA; t.width = d.d_out; t.ldx = t.ldy = d.d_out;
      t.in_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(t, s));
      COFREE_TRY(together ? launch_wgrads(u, ua, sums, s) : launch_wgrad(ua, sums, s));
      GemmArgs z = gemm();
      z.A1 = p.dA; z.lda1 = d.d_out; z.K1 = d.d_out;
      z.B = params->U; z.ldb = ldu; z.b_kmajor = 1;
      z.C = p.dZ; z.ldc = d.d_msg; z.N = d.d_msg;
      z.gate = Z; z.ldg = d.d_msg;
      COFREE_TRY(launch_gemm(z, s));
    } else {
      // dU_a = dP^T A (side stream as well)
      COFREE_TRY(merged_dU ? launch_wgrad(u, sums, s2)
                           : launch_wgrads(u, wgrad(dP, d.d_out, A, d.d_msg, grads->U, ldu, p.wg[1]), sums, s2));
      // dA / deg = (dP U_a) scaled per destination row, so that the transposed mean is a plain pull
      GemmArgs a = gemm();
      a.A1 = dP; a.lda1 = d.d_out; a.K1 = d.d_out;
      a.B = params->U; a.ldb = ldu; a.b_kmajor = 1;
      a.C = p.dA; a.ldc = d.d_msg; a.N = d.d_msg;
      a.row_scale = g.inv_deg;
      COFREE_TRY(launch_gemm(a, s));
      // dZ[u] = [Z[u] > 0] * sum_{v in N(u)} dA[v] / deg(v)
      AggArgs t = agg();
      t.X = p.dA; t.Y = p.dZ; t.width = d.d_msg; t.ldx = t.ldy = d.d_msg;
      t.relu_src = Z; t.ld_relu = d.d_msg;
      COFREE_TRY(launch_aggregate(t, s));
    }
    // dW = dZ^T H, dbW = column sums of dZ
    WgradArgs w = wgrad(p.dZ, d.d_msg, H_in, d.d_in, grads->W, d.d_in, p.wg[2]);
    w.colsum_out = grads->bW;
    COFREE_TRY(launch_wgrad(w, sums, s));
    if (dH_in) {
      // dH = dP U_s + dZ W: one product over the two k-segments [dP | dZ], each with its own parameters
      GemmArgs h = gemm();
      h.A1 = dP; h.lda1 = d.d_out; h.K1 = d.d_out;
      h.B = params->U + d.d_msg; h.ldb = ldu; h.b_kmajor = 1;
      h.A2 = p.dZ; h.lda2 = d.d_msg; h.K2 = d.d_msg;
      h.B2 = params->W; h.ldb2 = d.d_in;
      h.C = dH_in; h.ldc = d.d_in; h.N = d.d_in;
      COFREE_TRY(launch_gemm(h, s));
    }
    return joiner.finish();
  }

  // GCN and conventional GraphSAGE: dPre = dH_out gated by the activation and the dropout mask
  // (nothing to do when the layer above has applied both: COFREE_GRAD_OUT_GATED)
  const bool out_gated = (d.grad_flags & COFREE_GRAD_OUT_GATED) != 0;
  // ReLU / dropout backward of the layer below, carried by the kernel that writes dH_in
  const void* in_gate = (d.grad_flags & COFREE_GRAD_IN_GATED) ? H_in : nullptr;
  const float in_scale = 1.0f / (1.0f - d.dropout_q_below);  // inverted dropout of the layer below
  const void* dPre = dH_out;
  if ((d.dropout_q > 0.f || d.act) && !out_gated) {
    COFREE_TRY(launch_mask_grad(dt, dH_out, d.act ? H_out : nullptr, p.dP, n, d.d_out, dropout_of(d), s));
    dPre = p.dP;
  }
  SideStream* side = nullptr;
  hipStream_t s2 = fork_side(s, &side);
  SideJoin joiner{s, side};
  if (d.kind == COFREE_SAGE_CONV) {
    const int64_t ldw = 2 * (int64_t)d.d_in;
    // dW_self = dPre^T H and db = column sums of dPre need only dPre: side stream.  Aggregate-first layers
    // also have dW_neigh = dPre^T M, in the same launch where the widths allow it
    const bool merged_dW = conv_merged(d);
    WgradArgs w = wgrad(dPre, d.d_out, H_in, d.d_in, grads->W, ldw, p.wg[0]);
    if (merged_dW) {
      COFREE_REQUIRE(saved->A, "layer_bwd: saved.A is NULL");
      w.B2 = saved->A, w.ldb2 = w.N2b = d.d_in;
    }
    w.colsum_out = grads->bW;
    const bool transform_first = conv_transform_first(d);
    if (!transform_first) COFREE_REQUIRE(saved->A, "layer_bwd: saved.A is NULL");
    // dW_neigh = dT^T H where the forward pass was mean(H W_neigh^T), in the launch of dW_self where both can be:
    const WgradArgs wn = transform_first ? wgrad(p.T, d.d_out, H_in, d.d_in, grads->W + d.d_in, ldw, p.wg[1]) : WgradArgs{};
    // ... as two results of one product; with a second stream dW_self runs there beside the aggregation that dW_neigh waits for
    const bool both = !side && conv_two_wgrads(d, n);
    if (both) w.A2 = p.T, w.C2 = grads->W + d.d_in;
    const bool together = transform_first && !both && !side && wgrads_pair(w, wn);
    // dW_neigh = dPre^T M where the forward pass has kept M = mean(H) (side stream as well)
    if (!transform_first && !merged_dW)
      COFREE_TRY(launch_wgrads(w, wgrad(dPre, d.d_out, saved->A, d.d_in, grads->W + d.d_in, ldw, p.wg[1]), sums, s2));
    else if (!together && !both)
      COFREE_TRY(launch_wgrad(w, sums, s2));
    if (transform_first || (dH_in && conv_gathers_grad(d))) {
      AggArgs t = agg();  // dT = mean^T(dPre)
      t.X = dPre; t.Y = p.T; t.width = d.d_out; t.ldx = t.ldy = d.d_out;
      t.in_scale = g.inv_deg;
      COFREE_TRY(launch_aggregate(t, s));
      if (transform_first) COFREE_TRY(both ? launch_wgrad(w, sums, s) : together ? launch_wgrads(w, wn, sums, s) : launch_wgrad(wn, sums, s));
      if (dH_in) {
        GemmArgs h = gemm();
        // W_self and W_neigh are column blocks of W: dH = dT W_neigh + dPre W_self is one product over the
        // two k-segments [dT | dPre], each with its own block; the means first, which are the smaller terms
        h.A1 = p.T; h.lda1 = d.d_out; h.K1 = d.d_out;
        h.B = params->W + d.d_in; h.ldb = ldw; h.b_kmajor = 1;
        h.A2 = dPre; h.lda2 = d.d_out; h.K2 = d.d_out;
        h.B2 = params->W; h.ldb2 = ldw;
        h.C = dH_in; h.ldc = d.d_in; h.N = d.d_in;
        h.gate = in_gate; h.ldg = d.d_in; h.gate_scale = in_scale;
        COFREE_TRY(launch_gemm(h, s));
      }
    } else if (dH_in) {
      // dH = dPre W_self + mean^T(dPre W_neigh)
      GemmArgs h = gemm();
      h.A1 = dPre; h.lda1 = d.d_out; h.K1 = d.d_out;
      h.B = params->W + d.d_in; h.ldb = ldw; h.b_kmajor = 1;
      h.C = p.T; h.ldc = d.d_in; h.N = d.d_in;
      h.row_scale = g.inv_deg;  // scaled per destination row, so that the transposed mean is a plain pull
      COFREE_TRY(launch_gemm(h, s));
      AggArgs a = agg();
      a.X = p.T; a.Y = dH_in; a.width = d.d_in; a.ldx = a.ldy = d.d_in;
      COFREE_TRY(launch_aggregate(a, s));
      GemmArgs self = gemm();
      self.A1 = dPre; self.lda1 = d.d_out; self.K1 = d.d_out;
      self.B = params->W; self.ldb = ldw; self.b_kmajor = 1;
      self.C = dH_in; self.ldc = d.d_in; self.N = d.d_in;
      self.accumulate = 1;
      self.gate = in_gate; self.ldg = d.d_in; self.gate_last = 1; self.gate_scale = in_scale;
      COFREE_TRY(launch_gemm(self, s));
    }
    return joiner.finish();
  }
  if (gcn_transform_first(d)) {
    // forward was Ahat (H W^T): dT = Ahat dPre, dW = dT^T H, dH = dT W
    AggArgs a = agg();
    a.X = dPre; a.Y = p.T; a.width = d.d_out; a.ldx = a.ldy = d.d_out;
    a.in_scale = g.gcn_norm; a.out_scale = g.gcn_norm; a.self_loop = 1;
    COFREE_TRY(launch_aggregate(a, s));
    WgradArgs w = wgrad(p.T, d.d_out, H_in, d.d_in, grads->W, d.d_in, p.wg[0]);
    w.colsum_out = grads->bW;  // db = column sums of dPre, which dW does not read
    w.colsum_src = dPre;
    w.colsum_workspace = p.cs;
    COFREE_TRY(launch_wgrad(w, sums, s));
    if (dH_in) {
      GemmArgs h = gemm();
      h.A1 = p.T; h.lda1 = d.d_out; h.K1 = d.d_out;
      h.B = params->W; h.ldb = d.d_in; h.b_kmajor = 1;
      h.C = dH_in; h.ldc = d.d_in; h.N = d.d_in;
      h.gate = in_gate; h.ldg = d.d_in; h.gate_scale = in_scale;
      COFREE_TRY(launch_gemm(h, s));
    }
  } else {
    // forward was (Ahat H) W^T: dW = dPre^T (Ahat H), dH = Ahat (dPre W)
    COFREE_REQUIRE(saved->A, "layer_bwd: saved.A is NULL");
    WgradArgs w = wgrad(dPre, d.d_out, saved->A, d.d_in, grads->W, d.d_in, p.wg[0]);
    w.colsum_out = grads->bW;
    COFREE_TRY(launch_wgrad(w, sums, s2));
    if (dH_in) {
      GemmArgs h = gemm();
      h.A1 = dPre; h.lda1 = d.d_out; h.K1 = d.d_out;
      h.B = params->W; h.ldb = d.d_in; h.b_kmajor = 1;
      h.C = p.T; h.ldc = d.d_in; h.N = d.d_in;
      h.row_scale = g.gcn_norm;
      COFREE_TRY(launch_gemm(h, s));
      AggArgs a = agg();
      a.X = p.T; a.Y = dH_in; a.width = d.d_in; a.ldx = a.ldy = d.d_in;
      a.out_scale = g.gcn_norm; a.self_loop = 1;
      a.relu_src = in_gate; a.ld_relu = d.d_in; a.gate_scale = in_scale;
      COFREE_TRY(launch_aggregate(a, s));
    }
  }
  return joiner.finish();
}

extern "C" {

int32_t cofree_layer_bwd(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                         const cofree_layer_desc* desc, const void* H_in, const void* H_out,
                         const cofree_layer_params* params, const cofree_layer_saved* saved, const void* dH_out,
                         void* dH_in, const cofree_layer_grads* grads, int32_t accumulate, void* workspace,
                         size_t workspace_bytes, void* stream) {
  SplitSums sums;
  sums.accumulate = accumulate ? 1 : 0;
  COFREE_TRY(layer_bwd(part, masks, mask_id, desc, H_in, H_out, params, saved, dH_out, dH_in, grads, workspace, workspace_bytes,
                       nullptr, &sums, (hipStream_t)stream));
  return launch_split_sums(sums, (hipStream_t)stream);
}

size_t cofree_layers_workspace_bytes(const cofree_layer_desc* descs, int32_t n_layers, int64_t n_nodes) {
  if (!descs || n_layers < 1 || n_nodes < 0) return 0;
  size_t b = 256;
  for (int32_t l = 0; l < n_layers; ++l)
    b = max3(b, plan_fwd(descs[l], n_nodes, nullptr, SIZE_MAX).bytes, bwd_bytes(descs[l], n_nodes));
  const Deferral f = plan_deferral(n_layers, n_nodes, [&](int32_t l) { return descs[l]; });
  return f.worth ? max2(b, f.scratch + f.partials) : b;
}

int32_t cofree_layers_fwd(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                          const cofree_layer_call* layers, int32_t n_layers, void* workspace, size_t workspace_bytes,
                          void* stream) {
  COFREE_REQUIRE(n_layers >= 0 && (n_layers == 0 || layers), "layers_fwd: bad layer list");
  for (int32_t l = 0; l < n_layers; ++l) {
    const cofree_layer_call& c = layers[l];
    COFREE_TRY(cofree_layer_fwd(part, masks, mask_id, &c.desc, c.H_in, &c.params, c.H_out, &c.saved, workspace,
                                workspace_bytes, stream));
  }
  return COFREE_OK;
}

int32_t cofree_layers_bwd(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                          const cofree_layer_call* layers, int32_t n_layers, int32_t accumulate, void* workspace,
                          size_t workspace_bytes, void* stream) {
  COFREE_REQUIRE(n_layers >= 0 && (n_layers == 0 || layers), "layers_bwd: bad layer list");
  if (n_layers == 0) return COFREE_OK;
  hipStream_t s = (hipStream_t)stream;
  for (int32_t l = 0; l < n_layers; ++l) COFREE_TRY(check_desc(&layers[l].desc));
  DeviceGraph g;
  COFREE_TRY(select_graph(part, masks, mask_id, &g));
  const Deferral f = plan_deferral(n_layers, g.n, [&](int32_t l) { return layers[l].desc; });
  const bool defer = f.worth && workspace && workspace_bytes >= f.scratch + f.partials;
  Carver partials(defer ? (char*)workspace + f.scratch : nullptr);
  SplitSums sums;
  sums.accumulate = accumulate ? 1 : 0;
  int32_t rc = COFREE_OK;
  for (int32_t l = n_layers - 1; l >= 0 && rc == COFREE_OK; --l) {
    const cofree_layer_call& c = layers[l];
    const int32_t before = sums.n;
    rc = layer_bwd(part, masks, mask_id, &c.desc, c.H_in, c.H_out, &c.params, &c.saved, c.dH_out, c.dH_in, &c.grads, workspace,
                   workspace_bytes, defer ? &partials : nullptr, &sums, s);
    if (rc != COFREE_OK) sums.n = before;
    COFREE_TRY(sums_of_one_launch(&sums, before, s));  // layers that share a gradient are summed one after the other
    if (defer && l > 0 && rc == COFREE_OK && sums.n + SplitSums::PER_LAYER <= SplitSums::MAX) continue;
    COFREE_TRY(launch_split_sums(sums, s));
    sums.n = 0;
  }
  return rc;
}

}  // extern "C"
