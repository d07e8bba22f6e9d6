// C ABI of libsmoe: argument checks, workspace layout and the order of kernel launches for
// ParallelLinear (Alg. 1, Alg. 2) and the SMoE MLP (Alg. 3).  No entry point allocates,
// synchronises or touches the host copy of any tensor.
#include "common.h"
#include <new>

namespace {
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

bool routing_ok(const smoe_routing *r) {
  if (!r || r->Tk < 0 || r->E < 1 || !r->expert_offsets) return false;
  return r->Tk == 0 || (r->sorted_expert_idxs && r->sorted_scattered_idxs);  // empty index arrays may be null
}
// Row widths must allow 16-byte accesses in the row kernels.
bool width_ok(smoe_dtype dt, int d) { return d > 0 && d % (int)(16 / dtype_size(dt)) == 0; }
bool dtype_ok(int dt) { return dt == SMOE_F32 || dt == SMOE_BF16; }

// what every launch of the persistent kernels takes from the context
void set_launch(const smoe_ctx *ctx, S2SArgs &a) {
  a.grid = ctx->stream_grid;
  a.group_m = ctx->group_m;
  a.tile_shape = ctx->tile_shape;
  a.clock_probe = ctx->clock_probe;
}
int run_s2s(smoe_ctx *ctx, hipStream_t s, smoe_dtype dt, S2SArgs a) {
  set_launch(ctx, a);
  if (dt == SMOE_BF16 && ctx->kernel_mode == 0 && s2s_decode_supported(a)) return launch_s2s_decode(s, a);
  if (dt == SMOE_BF16 && ctx->kernel_mode == 0 && s2s_stream_supported(a)) return launch_s2s_stream(s, a);
  if (dt == SMOE_BF16 && ctx->kernel_mode != 1 && s2s_mfma_supported(a)) return launch_s2s_mfma(s, a);
  return launch_s2s_plain(s, dt, a);
}
int run_dw(smoe_ctx *ctx, hipStream_t s, smoe_dtype dt, DWArgs a) {
  a.grid = ctx->stream_grid;
  if (dt == SMOE_BF16 && ctx->kernel_mode == 0 && dw_stream_supported(a)) return launch_dw_stream(s, a);
  if (dt == SMOE_BF16 && ctx->kernel_mode != 1 && dw_mfma_supported(a)) return launch_dw_mfma(s, a);
  return launch_dw_plain(s, dt, a);
}
constexpr size_t SPREAD_MIN_ELEMENTS = (size_t)24 << 20;   // plinear_bwd says why

// Does the persistent groupXTY take these operands, rows that it reads through the order indices among them?
bool dw_reads_rows(const smoe_ctx *ctx, DWArgs a) {
  a.grid = ctx->stream_grid;
  return ctx->kernel_mode == 0 && dw_stream_supported(a);
}

// Do two arrays share memory?  (An output over an input that only an earlier launch reads is fine while these are launches of their
// own, and not where one launch does it all.)
bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes) {
  const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
  return a && b && p < q + b_bytes && q < p + a_bytes;
}
// The parts of an fp32 backward pass that wait for nothing but their inputs: in one launch, or (`apart`, or too many blocks for
// one) in the order row dots, weight gradient, input gradient.
int run_f32_backward(hipStream_t s, const S2SArgs &x, const DWArgs &w, const RowDots &d, bool apart) {
  if (!apart && f32_backward_fits(x, w, d)) return launch_f32_backward(s, x, w, d);
  int rc = d.dg ? launch_rowdot(s, SMOE_F32, d.dY, d.Yhat, d.dg, d.Tk, d.kp, d.d) : SMOE_OK;
  if (rc == SMOE_OK && w.dW) rc = launch_dw_plain(s, SMOE_F32, w);
  if (rc == SMOE_OK && x.C) rc = launch_s2s_plain(s, SMOE_F32, x);
  return rc;
}

S2SArgs make_s2s(const void *A, const void *W, void *C, const smoe_routing *r, int d_in, int d_out, bool trans_w,
                 bool a_grouped, int a_fan, bool c_grouped) {
  S2SArgs a;
  a.A = A; a.W = W; a.C = C;
  a.a_map = RowMap{a_grouped ? nullptr : r->sorted_scattered_idxs, a_fan};
  a.c_map = RowMap{c_grouped ? nullptr : r->sorted_scattered_idxs, 1};
  a.offsets = r->expert_offsets;
  a.E = r->E; a.Tk = r->Tk;
  a.K = trans_w ? d_out : d_in;
  a.N = trans_w ? d_in : d_out;
  a.ldw = d_out;
  a.w_stride = (size_t)d_in * d_out;
  a.trans_w = trans_w ? 1 : 0;
  a.H = nullptr;
  a.tail_ws = nullptr;
  return a;
}
}  // namespace

extern "C" {

int smoe_abi_version(void) { return 1; }

const char *smoe_strerror(int status) {
  switch (status) {
    case SMOE_OK: return "ok";
    case SMOE_ERR_INVALID_ARG: return "invalid argument";
    case SMOE_ERR_UNSUPPORTED: return "unsupported shape or option (row widths must be multiples of 16 bytes)";
    case SMOE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case SMOE_ERR_HIP: return "HIP runtime error";
    case SMOE_ERR_TOO_LARGE: return "problem exceeds the fixed scratch capacity of a no-allocation entry point";
    default: return "unknown status";
  }
}

int smoe_create(smoe_ctx **out, int device) {
  if (!out) return SMOE_ERR_INVALID_ARG;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess) return SMOE_ERR_HIP;
  if (device < 0 || device >= count) return SMOE_ERR_INVALID_ARG;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return SMOE_ERR_HIP;
  smoe_ctx *c = new (std::nothrow) smoe_ctx;
  if (!c) return SMOE_ERR_HIP;
  c->device = device;
  c->num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  // persistent kernels: one block per compute unit, dealt to the XCDs in eight equal shares
  c->stream_grid = c->num_cu >= 256 ? 256 : (c->num_cu & ~7);
  c->kernel_mode = 0;
  c->group_m = 4;
  c->tile_shape = 0;
  c->clock_probe = nullptr;
  c->route_scratch = nullptr;
  // kernel attributes and the address of a __device__ array are per device: set them with this context's device current, then restore the caller's
  int prev = -1;
  int rc = SMOE_ERR_HIP;
  if (hipGetDevice(&prev) == hipSuccess && hipSetDevice(device) == hipSuccess) {
    rc = init_stream_kernels();
    if (rc == SMOE_OK) rc = init_mfma_kernels();
    if (rc == SMOE_OK) rc = init_route_kernels();
    if (rc == SMOE_OK) rc = route_scratch_address(&c->route_scratch);
    if (hipSetDevice(prev) != hipSuccess && rc == SMOE_OK) rc = SMOE_ERR_HIP;
  }
  if (rc != SMOE_OK) {
    delete c;
    return rc;
  }
  *out = c;
  return SMOE_OK;
}

void smoe_destroy(smoe_ctx *ctx) { delete ctx; }

int smoe_set_kernel_mode(smoe_ctx *ctx, int mode) {
  if (!ctx || mode < 0 || mode > 4) return SMOE_ERR_INVALID_ARG;
  ctx->kernel_mode = mode > 2 ? 0 : mode;
  ctx->tile_shape = mode > 2 ? mode - 2 : 0;
  return SMOE_OK;
}

int smoe_set_tile_group(smoe_ctx *ctx, int group_m) {
  if (!ctx || group_m < 1 || group_m > 64) return SMOE_ERR_INVALID_ARG;
  ctx->group_m = group_m;
  return SMOE_OK;
}

int smoe_set_clock_probe(smoe_ctx *ctx, uint64_t *device_array) {
  if (!ctx) return SMOE_ERR_INVALID_ARG;
  ctx->clock_probe = (unsigned long long *)device_array;
  return SMOE_OK;
}

int smoe_topk_gate(smoe_ctx *ctx, void *stream, const float *logits, int T, int E, int k, int32_t *expert_idxs,
                   float *gates) {
  if (!ctx || T < 0 || E < 1 || k < 1 || k > E) return SMOE_ERR_INVALID_ARG;
  if (T == 0) return SMOE_OK;
  if (!logits || !expert_idxs || !gates) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k > 0x7fffffffLL) return SMOE_ERR_UNSUPPORTED;
  return launch_topk_gate((hipStream_t)stream, logits, T, E, k, expert_idxs, gates);
}

int smoe_topk_gate_bwd(smoe_ctx *ctx, void *stream, const int32_t *expert_idxs, const float *gates, const float *dgates,
                       int T, int E, int k, float *dlogits) {
  if (!ctx || T < 0 || E < 1 || k < 1 || k > E) return SMOE_ERR_INVALID_ARG;
  if (T == 0) return SMOE_OK;
  if (!expert_idxs || !gates || !dgates || !dlogits) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k > 0x7fffffffLL) return SMOE_ERR_UNSUPPORTED;
  return launch_topk_gate_bwd((hipStream_t)stream, expert_idxs, gates, dgates, T, E, k, dlogits);
}

static int attention_args_ok(smoe_dtype dtype, int B, int T, int G, int h, int d_head) {
  if (B < 1 || T < 1 || G < 1 || h < 1 || d_head < 1) return SMOE_ERR_INVALID_ARG;
  if (dtype != SMOE_BF16 || d_head != 128) return SMOE_ERR_UNSUPPORTED;
  if ((long long)T * G > 0x3fffffffLL || (long long)B * T * G > 0x7fffffffLL || h > 65535 || B > 65535)
    return SMOE_ERR_UNSUPPORTED;
  if ((((long long)T * G + 127) / 128) * h * B > 0x7fffffffLL) return SMOE_ERR_UNSUPPORTED;   // one-dimensional grids
  return SMOE_OK;
}

int smoe_attention_fwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *Q, const void *K, const void *V, int B,
                       int T, int G, int h, int d_head, void *O, float *LSE) {
  if (!ctx || !Q || !K || !V || !O || !LSE) return SMOE_ERR_INVALID_ARG;
  int rc = attention_args_ok(dtype, B, T, G, h, d_head);
  if (rc != SMOE_OK) return rc;
  return launch_attn_fwd((hipStream_t)stream, Q, K, V, O, LSE, B, T, G, h);
}

size_t smoe_attention_bwd_workspace_bytes(int B, int T, int G, int h) {
  if (B < 1 || T < 1 || G < 1 || h < 1) return 0;
  return align256(attn_bwd_workspace_bytes(B, T, G, h));
}

int smoe_attention_bwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *dO, const void *Q, const void *K,
                       const void *V, const void *O, const float *LSE, int B, int T, int G, int h, int d_head, void *dQ,
                       void *dK, void *dV, void *ws, size_t ws_bytes) {
  if (!ctx || !dO || !Q || !K || !V || !O || !LSE || !dQ || !dK || !dV) return SMOE_ERR_INVALID_ARG;
  int rc = attention_args_ok(dtype, B, T, G, h, d_head);
  if (rc != SMOE_OK) return rc;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < smoe_attention_bwd_workspace_bytes(B, T, G, h)) return SMOE_ERR_WORKSPACE;
  return launch_attn_bwd((hipStream_t)stream, Q, K, V, O, dO, LSE, ws, dQ, dK, dV, B, T, G, h);
}

size_t smoe_route_workspace_bytes(int T, int k, int E) {
  if (T < 0 || k < 1 || E < 1) return 0;
  return route_workspace_bytes(T * k, E);
}

int smoe_route(smoe_ctx *ctx, void *stream, const int32_t *expert_idxs, int T, int k, int E,
               int32_t *sorted_expert_idxs, int32_t *sorted_scattered_idxs, int32_t *expert_offsets, void *ws,
               size_t ws_bytes) {
  if (!ctx || T < 0 || k < 1 || E < 1 || !expert_offsets) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k > 0x7fffffffLL || E > ROUTE_MAX_E) return SMOE_ERR_UNSUPPORTED;
  if (T > 0 && (!expert_idxs || !sorted_expert_idxs || !sorted_scattered_idxs)) return SMOE_ERR_INVALID_ARG;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < route_workspace_bytes(T * k, E)) return SMOE_ERR_WORKSPACE;
  return launch_route((hipStream_t)stream, expert_idxs, T * k, E, sorted_expert_idxs, sorted_scattered_idxs,
                      expert_offsets, ws);
}

int smoe_route_noalloc(smoe_ctx *ctx, void *stream, const int32_t *expert_idxs, int T, int k, int E,
                       int32_t *sorted_expert_idxs, int32_t *sorted_scattered_idxs, int32_t *expert_offsets) {
  if (!ctx || T < 0 || k < 1 || E < 1 || !expert_offsets) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k > 0x7fffffffLL || E > ROUTE_MAX_E) return SMOE_ERR_UNSUPPORTED;
  if (T > 0 && (!expert_idxs || !sorted_expert_idxs || !sorted_scattered_idxs)) return SMOE_ERR_INVALID_ARG;
  if (route_workspace_bytes(T * k, E) > ROUTE_SCRATCH_BYTES) return SMOE_ERR_TOO_LARGE;
  if (!ctx->route_scratch) return SMOE_ERR_HIP;
  // Nothing in the scratch has to start at zero: the counting kernel writes every (expert, chunk) counter
  // before the scan reads it, and a one-chunk problem does not touch the scratch at all.
  return launch_route((hipStream_t)stream, expert_idxs, T * k, E, sorted_expert_idxs, sorted_scattered_idxs,
                      expert_offsets, ctx->route_scratch);
}

int smoe_group(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *in, int d, const smoe_routing *r, int fan,
               const float *gates, void *out) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || fan < 1 || d < 1) return SMOE_ERR_INVALID_ARG;
  if (r->Tk == 0) return SMOE_OK;
  if (!in || !out || r->Tk % fan) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d) || !aligned16(in) || !aligned16(out)) return SMOE_ERR_UNSUPPORTED;
  return launch_group((hipStream_t)stream, dtype, in, r->sorted_scattered_idxs, fan, gates, out, r->Tk, d);
}

// ------------------------------------------------------------------------------ Alg. 1
int smoe_plinear_fwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *X, int x_rows, int d_in,
                     const void *W, int d_out, const smoe_routing *r, int k, const float *gates, int gates_k,
                     int grouped_in, int grouped_out, void *Yhat, void *Y) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || d_in < 1 || d_out < 1 || k < 1 || x_rows < 0)
    return SMOE_ERR_INVALID_ARG;
  const int Tk = r->Tk;
  if (grouped_in ? (k != 1 || x_rows != Tk) : ((long long)x_rows * k != Tk)) return SMOE_ERR_INVALID_ARG;
  if (gates) {
    if (grouped_out || gates_k < 1 || Tk % gates_k || !Y) return SMOE_ERR_INVALID_ARG;
  } else if (Y) {
    return SMOE_ERR_INVALID_ARG;
  }
  if (Tk == 0) return SMOE_OK;
  if (!X || !W || !Yhat) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d_in) || !width_ok(dtype, d_out) || !aligned16(X) || !aligned16(W) || !aligned16(Yhat) ||
      (Y && !aligned16(Y)))
    return SMOE_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  S2SArgs a = make_s2s(X, W, Yhat, r, d_in, d_out, false, grouped_in != 0, k, grouped_out != 0);
  int rc = run_s2s(ctx, s, dtype, a);
  if (rc != SMOE_OK) return rc;
  if (gates) rc = launch_combine(s, dtype, Yhat, gates, Y, Tk / gates_k, gates_k, d_out);
  return rc;
}

// ------------------------------------------------------------------------------ Alg. 2
// Workspace: [dYbar: Tk x d_out, when dY arrives scattered (weighted or not) -- Alg. 2's group(dY, o, p)]
//            [Xbar:  Tk x d_in, when X was scattered -- Alg. 2's group(X, o); the same array then
//                    receives dXbar, the reuse Sec. 3.2.1 points out]
//            [64 MiB of fp32 partial tiles; before the first product they hold the inverse of the order indices]
static void plinear_bwd_layout(smoe_dtype dt, int d_in, int d_out, int Tk, int grouped_in, int grouped_out,
                               size_t &off_dybar, size_t &off_xbar, size_t &total) {
  size_t es = dtype_size(dt), off = 0;
  off_dybar = off_xbar = (size_t)-1;
  if (!grouped_out) { off_dybar = off; off += align256((size_t)Tk * d_out * es); }
  if (!grouped_in) { off_xbar = off; off += align256((size_t)Tk * d_in * es); }
  total = off + S2S_TAIL_WS_BYTES;   // fp32 partial tiles of the input-gradient product's split last round
}

size_t smoe_plinear_bwd_workspace_bytes(smoe_dtype dtype, int x_rows, int d_in, int d_out, int Tk, int k,
                                        int has_gates, int grouped_in, int grouped_out) {
  (void)x_rows; (void)k; (void)has_gates;
  if (!dtype_ok(dtype) || d_in < 1 || d_out < 1 || Tk < 0) return 0;
  size_t a, b, total;
  plinear_bwd_layout(dtype, d_in, d_out, Tk, grouped_in, grouped_out, a, b, total);
  return total;
}

// given_inv: the inverse of the order indices where the caller has it already (NULL: made here when it pays).
// more0, more1: two further contributions to dX [x_rows, d_in], added where the k slots are summed (scattered X with k > 1)
static int plinear_bwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *dY, const void *X, int x_rows,
                     int d_in, const void *W, int d_out, const void *Yhat, const smoe_routing *r, int k,
                     const float *gates, int gates_k, int grouped_in, int grouped_out, void *dX, void *dW,
                     float *dgates, void *ws, size_t ws_bytes, const void *more0, const void *more1, const int32_t *given_inv) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || d_in < 1 || d_out < 1 || k < 1 || x_rows < 0)
    return SMOE_ERR_INVALID_ARG;
  const int Tk = r->Tk;
  if (grouped_in ? (k != 1 || x_rows != Tk) : ((long long)x_rows * k != Tk)) return SMOE_ERR_INVALID_ARG;
  if (gates && (grouped_out || gates_k < 1 || Tk % gates_k)) return SMOE_ERR_INVALID_ARG;
  if (!gates && dgates) return SMOE_ERR_INVALID_ARG;
  if (dgates && !Yhat) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d_in) || !width_ok(dtype, d_out)) return SMOE_ERR_UNSUPPORTED;
  if (!W && dX) return SMOE_ERR_INVALID_ARG;
  size_t off_dybar, off_xbar, need;
  plinear_bwd_layout(dtype, d_in, d_out, Tk, grouped_in, grouped_out, off_dybar, off_xbar, need);
  if (need && (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)) return SMOE_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  int rc = SMOE_OK;
  if (Tk == 0) {  // no routed rows: dW is all zeros, nothing else to write
    if (dW) {
      DWArgs z{nullptr, nullptr, dW, r->expert_offsets, r->E, 0, d_in, d_out};
      rc = launch_dw_plain(s, dtype, z);
    }
    return rc;
  }
  if (!dY || !X) return SMOE_ERR_INVALID_ARG;
  if (!aligned16(dY) || !aligned16(X) || (W && !aligned16(W)) || (dX && !aligned16(dX)) || (dW && !aligned16(dW)))
    return SMOE_ERR_UNSUPPORTED;

  if (dtype == SMOE_F32) {
    // The fp32 kernels read the rows of dY and X through the order indices and apply the routing weights themselves: no
    // sorted copies, and no launches to make them.
    const RowDots d{dY, Yhat, gates ? dgates : nullptr, Tk, gates_k, d_out};
    const RowMap y_map{grouped_out ? nullptr : r->sorted_scattered_idxs, gates ? gates_k : 1};
    DWArgs w{X, dY, dW, r->expert_offsets, r->E, Tk, d_in, d_out};
    w.a_map = RowMap{grouped_in ? nullptr : r->sorted_scattered_idxs, k};
    w.b_map = y_map;
    w.gates = gates;
    const bool need_sum = !grouped_in && k > 1;
    void *dst = need_sum && dX ? (void *)((char *)ws + off_xbar) : dX;
    S2SArgs a = make_s2s(dY, W, dst, r, d_in, d_out, true, grouped_out != 0, y_map.fan, grouped_in != 0);
    a.gates = gates;
    a.slots = r->sorted_scattered_idxs;
    const size_t x_bytes = (size_t)x_rows * d_in * 4, w_bytes = (size_t)r->E * d_in * d_out * 4, dst_bytes = (size_t)Tk * d_in * 4;
    const size_t yhat_bytes = d.dg ? (size_t)Tk * d_out * 4 : 0;
    const bool apart = overlap(dst, dst_bytes, X, x_bytes) || overlap(dst, dst_bytes, Yhat, yhat_bytes) || overlap(dW, w_bytes, Yhat, yhat_bytes) || overlap(dst, dst_bytes, dgates, (size_t)Tk * 4) ||
                       overlap(dst, dst_bytes, dW, w_bytes) || overlap(dW, w_bytes, d.dg, (size_t)Tk * 4);
    rc = run_f32_backward(s, a, w, d, apart);
    if (rc != SMOE_OK || !need_sum || !dX) return rc;
    return launch_combine(s, dtype, dst, nullptr, dX, x_rows, k, d_in, more0, more1);
  }

  // dp = bmm(dY, Yhat); dYbar = group(dY, o, p)  (Alg. 2: "weight and group")
  int32_t *own_inv = (int32_t *)((char *)ws + need - S2S_TAIL_WS_BYTES);   // read before the first product writes partial tiles there
  const int32_t *inv = given_inv ? given_inv : own_inv;
  // Rows that several slots share are spread from the source rows when that saves more than the launch that inverts the order
  // indices costs (about 3 us): on 20500 rows of 3 and 4 KB 39 us of group copies became 28, on 8192 rows of 2 KB the launch was
  // dearer by 1.5 us, so from 24 Mi elements on.
  // groupXTY reads scattered rows of X, and of dY where no weights go with them, through the order indices: no sorted copy (unless an
  // output that is written meanwhile lies over them).  The input-gradient product gathers such rows of dY as well.
  const size_t x_bytes = (size_t)x_rows * d_in * 2, y_bytes = (size_t)Tk * d_out * 2, w_bytes = (size_t)r->E * d_in * d_out * 2;
  DWArgs w{X, dY, dW, r->expert_offsets, r->E, Tk, d_in, d_out};
  if (!grouped_in && !overlap(dW, w_bytes, X, x_bytes)) w.a_map = RowMap{r->sorted_scattered_idxs, k};
  const bool rows_x = w.a_map.o && dw_reads_rows(ctx, w);
  if (!rows_x) w.a_map = RowMap{nullptr, 1};
  if (!grouped_out && !gates && !overlap(dW, w_bytes, dY, y_bytes) && !overlap(dX, x_bytes, dY, y_bytes)) w.b_map = RowMap{r->sorted_scattered_idxs, 1};
  const bool rows_y = w.b_map.o && dw_reads_rows(ctx, w);
  if (!rows_y) w.b_map = RowMap{nullptr, 1};
  size_t shared = 0;
  if (!grouped_out && gates && gates_k > 1) shared += (size_t)Tk * d_out;
  if (!grouped_in && dW && k > 1 && !rows_x) shared += (size_t)Tk * d_in;
  const bool spread = given_inv || (shared >= SPREAD_MIN_ELEMENTS && (size_t)Tk * sizeof(int32_t) <= S2S_TAIL_WS_BYTES);
  const bool spread_y = spread && gates && gates_k > 1, spread_x = spread && k > 1 && !rows_x;
  if (spread && !given_inv) {
    rc = launch_invert(s, r->sorted_scattered_idxs, own_inv, Tk);
    if (rc != SMOE_OK) return rc;
  }
  void *xbar = grouped_in ? nullptr : (void *)((char *)ws + off_xbar);
  const bool spread_both = spread_y && spread_x && !grouped_in && dW && gates_k == k;
  const void *dYbar = dY;
  if (!grouped_out && !rows_y) {
    const RowDots dots{dY, Yhat, gates ? dgates : nullptr, Tk, gates_k, d_out};
    if (dots.dg && !spread_y) {
      rc = launch_rowdot(s, dtype, dY, Yhat, dgates, Tk, gates_k, d_out);
      if (rc != SMOE_OK) return rc;
    }
    void *buf = (char *)ws + off_dybar;
    rc = spread_y ? launch_spread(s, dY, inv, gates_k, gates, buf, Tk, d_out, dots, spread_both ? X : nullptr, spread_both ? xbar : nullptr, d_in)
                  : launch_group(s, dtype, dY, r->sorted_scattered_idxs, gates ? gates_k : 1, gates, buf, Tk, d_out);
    if (rc != SMOE_OK) return rc;
    dYbar = buf;
  }
  // Xbar = group(X, o);  dW = groupXTY(Xbar, dYbar)
  if (dW) {
    if (!grouped_in && !rows_x) {
      rc = spread_both ? SMOE_OK : spread_x ? launch_spread(s, X, inv, k, nullptr, xbar, Tk, d_in)
                    : launch_group(s, dtype, X, r->sorted_scattered_idxs, k, nullptr, xbar, Tk, d_in);
      if (rc != SMOE_OK) return rc;
      w.A = xbar;
    }
    w.B = dYbar;
    w.split_ws = (float *)((char *)ws + need - S2S_TAIL_WS_BYTES);   // the input-gradient product below uses it afterwards
    rc = run_dw(ctx, s, dtype, w);
    if (rc != SMOE_OK) return rc;
  }
  // dXbar = scatter2scatter(dYbar, W^T, o, 1): grouped or scattered like the forward input;
  // with fan-out k the k slot gradients of a row are then summed.
  if (dX) {
    bool need_sum = !grouped_in && k > 1;
    void *dst = need_sum ? xbar : dX;   // Xbar is dead once dW is done
    S2SArgs a = make_s2s(dYbar, W, dst, r, d_in, d_out, true, !rows_y, 1, grouped_in != 0);
    a.tail_ws = (float *)((char *)ws + need - S2S_TAIL_WS_BYTES);
    rc = run_s2s(ctx, s, dtype, a);
    if (rc != SMOE_OK) return rc;
    if (need_sum) rc = launch_combine(s, dtype, dst, nullptr, dX, x_rows, k, d_in, more0, more1);
  }
  return rc;
}

int smoe_plinear_bwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *dY, const void *X, int x_rows,
                     int d_in, const void *W, int d_out, const void *Yhat, const smoe_routing *r, int k,
                     const float *gates, int gates_k, int grouped_in, int grouped_out, void *dX, void *dW,
                     float *dgates, void *ws, size_t ws_bytes) {
  return plinear_bwd(ctx, stream, dtype, dY, X, x_rows, d_in, W, d_out, Yhat, r, k, gates, gates_k, grouped_in, grouped_out, dX, dW, dgates,
                     ws, ws_bytes, nullptr, nullptr, nullptr);
}

// ------------------------------------------------------------------------------ Alg. 3
static inline int hidden_width(smoe_act act, int d_expert) { return act == SMOE_ACT_SWIGLU ? 2 * d_expert : d_expert; }

// Hpre = ParallelLinear(X, W1, scattered -> grouped);  H = sigma(Hpre)   (first two lines of Alg. 3).
// Hpre always points at room for the pre-activation; keep_hpre says whether the caller wants it written
// (when the activation is applied in the product's epilogue it is otherwise never stored).
static int hidden_forward(smoe_ctx *ctx, hipStream_t s, smoe_dtype dtype, smoe_act act, const void *X, int d_model,
                          int d_expert, const void *W1, const smoe_routing *r, int k, void *Hpre, bool keep_hpre, void *H,
                          float *tail_ws, size_t call_weights) {
  const int d_h = hidden_width(act, d_expert);
  S2SArgs a1 = make_s2s(X, W1, Hpre, r, d_model, d_h, false, false, k, true);
  a1.tail_ws = tail_ws;
  a1.call_weights = call_weights;
  S2SArgs fused = a1;
  fused.H = H;
  set_launch(ctx, fused);
  if (act == SMOE_ACT_SWIGLU && dtype == SMOE_BF16 && ctx->kernel_mode == 0 &&
      (s2s_decode_supported(fused) || s2s_stream_swiglu_supported(fused))) {
    // SwiGLU in the product's epilogue: H comes straight from the fp32 accumulators, and the
    // pre-activation is written only when the caller keeps it for the backward pass
    if (!keep_hpre) fused.C = nullptr;
    return s2s_decode_supported(fused) ? launch_s2s_decode(s, fused) : launch_s2s_stream(s, fused);
  }
  if (dtype == SMOE_F32) {   // the fp32 kernels apply any activation in the epilogue
    a1.H = H;
    a1.act = act;
    if (!keep_hpre) a1.C = nullptr;
    return launch_s2s_plain(s, dtype, a1);
  }
  int rc = run_s2s(ctx, s, dtype, a1);
  if (rc != SMOE_OK) return rc;
  return launch_act_fwd(s, act, Hpre, H, r->Tk, d_expert);
}

size_t smoe_plinear_act_fwd_workspace_bytes(smoe_dtype dtype, smoe_act act, int T, int k, int d_model, int d_expert,
                                            int keep_hpre) {
  if (!dtype_ok(dtype) || T < 0 || k < 1 || d_model < 1 || d_expert < 1) return 0;
  size_t hpre = keep_hpre ? 0 : align256((size_t)T * k * hidden_width(act, d_expert) * dtype_size(dtype));
  return hpre + S2S_TAIL_WS_BYTES;
}

int smoe_plinear_act_fwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, smoe_act act, const void *X, int T, int d_model,
                         int d_expert, const void *W1, const smoe_routing *r, int k, void *Hpre, void *H, void *ws,
                         size_t ws_bytes) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || T < 0 || k < 1 || d_model < 1 || d_expert < 1)
    return SMOE_ERR_INVALID_ARG;
  if (act != SMOE_ACT_NONE && act != SMOE_ACT_GELU && act != SMOE_ACT_SWIGLU) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k != r->Tk) return SMOE_ERR_INVALID_ARG;
  if (T == 0) return SMOE_OK;
  if (!X || !W1 || !H) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d_model) || !width_ok(dtype, d_expert)) return SMOE_ERR_UNSUPPORTED;
  size_t need = smoe_plinear_act_fwd_workspace_bytes(dtype, act, T, k, d_model, d_expert, Hpre != nullptr);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return SMOE_ERR_WORKSPACE;
  float *tail_ws = (float *)((char *)ws + need - S2S_TAIL_WS_BYTES);
  void *pre = Hpre ? Hpre : ws;
  if (!aligned16(X) || !aligned16(W1) || !aligned16(H) || !aligned16(pre)) return SMOE_ERR_UNSUPPORTED;
  return hidden_forward(ctx, (hipStream_t)stream, dtype, act, X, d_model, d_expert, W1, r, k, pre, Hpre != nullptr, H, tail_ws, 0);
}

size_t smoe_mlp_fwd_workspace_bytes(smoe_dtype dtype, smoe_act act, int T, int k, int d_model, int d_expert,
                                    int training) {
  if (!dtype_ok(dtype) || T < 0 || k < 1 || d_model < 1 || d_expert < 1) return 0;
  size_t es = dtype_size(dtype), Tk = (size_t)T * k;
  if (training == 1) return S2S_TAIL_WS_BYTES;
  if (training == 2) return align256(Tk * d_model * es) + S2S_TAIL_WS_BYTES;      // Hpre and H kept, Yhat lives here
  return align256(Tk * hidden_width(act, d_expert) * es) + align256(Tk * d_expert * es) +
         align256(Tk * d_model * es) + S2S_TAIL_WS_BYTES;
}

int smoe_mlp_fwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, smoe_act act, const void *X, int T, int d_model,
                 int d_expert, const void *W1, const void *W2, const smoe_routing *r, int k, const float *gates,
                 void *Y, void *saved_Hpre, void *saved_H, void *saved_Yhat, void *ws, size_t ws_bytes) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || T < 0 || k < 1 || d_model < 1 || d_expert < 1)
    return SMOE_ERR_INVALID_ARG;
  if (act != SMOE_ACT_NONE && act != SMOE_ACT_GELU && act != SMOE_ACT_SWIGLU) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k != r->Tk) return SMOE_ERR_INVALID_ARG;
  const int nhid = (saved_Hpre != nullptr) + (saved_H != nullptr);
  if (nhid == 1 || (nhid == 0 && saved_Yhat)) return SMOE_ERR_INVALID_ARG;
  const int nsaved = nhid ? 3 : 0;                      // 3: training (Yhat may still live in the workspace)
  const int mode = nhid == 0 ? 0 : (saved_Yhat ? 1 : 2);
  if (T == 0) return SMOE_OK;
  if (!X || !W1 || !W2 || !gates || !Y) return SMOE_ERR_INVALID_ARG;
  const int d_h = hidden_width(act, d_expert), Tk = r->Tk;
  if (!width_ok(dtype, d_model) || !width_ok(dtype, d_expert)) return SMOE_ERR_UNSUPPORTED;
  size_t es = dtype_size(dtype);
  size_t need = smoe_mlp_fwd_workspace_bytes(dtype, act, T, k, d_model, d_expert, mode);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return SMOE_ERR_WORKSPACE;
  float *tail_ws = (float *)((char *)ws + need - S2S_TAIL_WS_BYTES);   // partial tiles of a split last round
  if (mode == 2) saved_Yhat = ws;
  if (nsaved == 0) {
    saved_Hpre = ws;
    saved_H = (char *)saved_Hpre + align256((size_t)Tk * d_h * es);
    saved_Yhat = (char *)saved_H + align256((size_t)Tk * d_expert * es);
  }
  if (!aligned16(X) || !aligned16(W1) || !aligned16(W2) || !aligned16(Y) || !aligned16(saved_Hpre) ||
      !aligned16(saved_H) || !aligned16(saved_Yhat))
    return SMOE_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  const size_t call_weights = (size_t)r->E * d_model * (d_h + d_expert) * es;
  int rc = hidden_forward(ctx, s, dtype, act, X, d_model, d_expert, W1, r, k, saved_Hpre, nsaved != 0, saved_H, tail_ws, call_weights);
  if (rc != SMOE_OK) return rc;
  // Y = ParallelLinear(H, W2, p, grouped -> scattered)
  S2SArgs a2 = make_s2s(saved_H, W2, saved_Yhat, r, d_expert, d_model, false, true, 1, false);
  a2.tail_ws = tail_ws;
  a2.call_weights = call_weights;
  rc = run_s2s(ctx, s, dtype, a2);
  if (rc != SMOE_OK) return rc;
  return launch_combine(s, dtype, saved_Yhat, gates, Y, T, k, d_model);
}

// Workspace of the backward pass: dYbar [Tk,d_model] (later reused for dXbar), dH [Tk,d_expert],
// dHpre [Tk,d_h].
// Backward passes that form dp in the epilogue of the W2^T product (bf16 through the persistent kernels).
// That product gathers the rows of dY itself, and groupXTY those of X, and of dY where the routing weights go with the hidden rows.
//   mode 1 (SwiGLU): the activation's derivative is applied there too; scratch = one array [Tk,d_model], dHpre [Tk,d_h].  The array
//     holds the routing-weighted hidden rows Hw [Tk,d_expert] where they are no wider, else the weighted sorted copy of dY.
//   mode 2 (other activations): dp from the saved H; scratch = the same array or, when d_expert < d_model, one for Hw and one for
//     the plain sorted copy of dY that groupXTY may need beside it; dH [Tk,d_expert]; dHpre [Tk,d_h].
//   both: room for the inverse of the order indices [Tk] and the slabs of dp [Tk, 2 * ceil(d_expert / 256)] fp32.
// The array of dY's copy later holds dXbar (and before it Xbar, where a sorted copy of X is made).  The inverse of the order indices
// sits where the slabs come to lie while dY is spread, and, written by the kernel that adds the slabs, in its own room while X is.
struct MlpBwdEpiLayout {
  size_t dybar_u, second, dh, dhpre, inv_x, dp_part, total;
  int part_ld;
  bool use_hw;
};
static MlpBwdEpiLayout mlp_bwd_epi_layout(int mode, size_t es, size_t Tk, int d_model, int d_expert, int d_h) {
  MlpBwdEpiLayout L;
  size_t off = 0;
  L.part_ld = 2 * ceil_div(d_expert, 256);
  L.use_hw = mode == 2 && d_expert < d_model;
  L.dybar_u = off;  off += L.use_hw ? align256(Tk * d_model * es) : 0;
  L.second = off;   off += align256(Tk * (size_t)(L.use_hw ? d_expert : d_model) * es);
  L.dh = off;       off += mode == 2 ? align256(Tk * (size_t)d_expert * es) : 0;
  L.dhpre = off;    off += align256(Tk * (size_t)d_h * es);
  L.inv_x = off;    off += align256(Tk * sizeof(int32_t));
  L.dp_part = off;  off += align256(Tk * (size_t)L.part_ld * sizeof(float));
  L.total = off + S2S_TAIL_WS_BYTES;
  return L;
}

size_t smoe_mlp_bwd_workspace_bytes(smoe_dtype dtype, smoe_act act, int T, int k, int d_model, int d_expert) {
  if (!dtype_ok(dtype) || T < 0 || k < 1 || d_model < 1 || d_expert < 1) return 0;
  size_t es = dtype_size(dtype), Tk = (size_t)T * k;
  const int d_h = hidden_width(act, d_expert);
  size_t plain = align256(Tk * d_model * es) + align256(Tk * d_expert * es) + align256(Tk * d_h * es) + S2S_TAIL_WS_BYTES;
  if (dtype != SMOE_BF16) return plain;
  size_t epi = mlp_bwd_epi_layout(act == SMOE_ACT_SWIGLU ? 1 : 2, es, Tk, d_model, d_expert, d_h).total;
  return epi > plain ? epi : plain;   // whichever path the shape takes fits
}

// How the backward pass of this shape runs: 0 = Alg. 2 step by step (dp from the forward's saved Yhat), 1 / 2 = dp in the
// epilogue of the W2^T product as described above (the forward's unweighted Yhat is then not needed).
static int mlp_bwd_mode(const smoe_ctx *ctx, smoe_dtype dtype, smoe_act act, int Tk, int k, int E, int d_model, int d_expert) {
  if (dtype != SMOE_BF16 || ctx->kernel_mode != 0 || Tk < 1) return 0;
  S2SArgs x;
  x.A = x.W = nullptr;  x.C = nullptr;
  x.a_map = RowMap{(const int32_t *)1, k};  x.c_map = RowMap{nullptr, 1};   // the product gathers the rows of dY [T, d_model]
  x.offsets = nullptr;  x.E = E;  x.Tk = Tk;
  x.K = d_model;  x.N = d_expert;  x.ldw = d_model;  x.w_stride = (size_t)d_expert * d_model;  x.trans_w = 1;
  x.tail_ws = nullptr;  x.H = nullptr;
  x.grid = ctx->stream_grid;
  x.row_scale = (const float *)1;  x.dp_part = (float *)1;   // only tested for presence
  if (act == SMOE_ACT_SWIGLU) {
    x.Hpre_in = (const void *)1;
    return s2s_stream_swiglu_bwd_supported(x) ? 1 : 0;
  }
  x.H_in = (const void *)1;
  return s2s_stream_dp_supported(x) ? 2 : 0;
}

int smoe_mlp_saves_yhat(smoe_ctx *ctx, smoe_dtype dtype, smoe_act act, int T, int k, int E, int d_model, int d_expert) {
  if (!ctx || !dtype_ok(dtype) || T < 0 || k < 1 || E < 1 || d_model < 1 || d_expert < 1) return SMOE_ERR_INVALID_ARG;
  return mlp_bwd_mode(ctx, dtype, act, T * k, k, E, d_model, d_expert) ? 0 : 1;
}

int smoe_mlp_bwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, smoe_act act, const void *dY, const void *X, int T,
                 int d_model, int d_expert, const void *W1, const void *W2, const smoe_routing *r, int k,
                 const float *gates, const void *saved_Hpre, const void *saved_H, const void *saved_Yhat, void *dX,
                 void *dW1, void *dW2, float *dgates, void *ws, size_t ws_bytes) {
  if (!ctx || !dtype_ok(dtype) || !routing_ok(r) || T < 0 || k < 1 || d_model < 1 || d_expert < 1)
    return SMOE_ERR_INVALID_ARG;
  if (act != SMOE_ACT_NONE && act != SMOE_ACT_GELU && act != SMOE_ACT_SWIGLU) return SMOE_ERR_INVALID_ARG;
  if ((long long)T * k != r->Tk) return SMOE_ERR_INVALID_ARG;
  if (!dW1 || !dW2) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d_model) || !width_ok(dtype, d_expert)) return SMOE_ERR_UNSUPPORTED;
  const int d_h = hidden_width(act, d_expert), Tk = r->Tk;
  size_t es = dtype_size(dtype);
  size_t need = smoe_mlp_bwd_workspace_bytes(dtype, act, T, k, d_model, d_expert);
  if (need && (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)) return SMOE_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  int rc = SMOE_OK;
  if (T == 0) {
    DWArgs z1{nullptr, nullptr, dW1, r->expert_offsets, r->E, 0, d_model, d_h};
    rc = launch_dw_plain(s, dtype, z1);
    if (rc != SMOE_OK) return rc;
    DWArgs z2{nullptr, nullptr, dW2, r->expert_offsets, r->E, 0, d_expert, d_model};
    return launch_dw_plain(s, dtype, z2);
  }
  const int mode = mlp_bwd_mode(ctx, dtype, act, Tk, k, r->E, d_model, d_expert);
  if (!dY || !X || !W1 || !W2 || !gates || !saved_Hpre || !saved_H || (!saved_Yhat && !mode) || !dX || !dgates)
    return SMOE_ERR_INVALID_ARG;
  if (!aligned16(dY) || !aligned16(X) || !aligned16(W1) || !aligned16(W2) || !aligned16(saved_Hpre) ||
      !aligned16(saved_H) || (saved_Yhat && !aligned16(saved_Yhat)) || !aligned16(dX) || !aligned16(dW1) || !aligned16(dW2))
    return SMOE_ERR_UNSUPPORTED;
  if (mode) {
    // Alg. 2 for both ParallelLinears with dp taken in the epilogue of the W2^T product: that product runs on the
    // UNWEIGHTED rows of dY, so its fp32 accumulators are dH / p and dp[row] = <acc, H[row]> needs neither the
    // forward's Yhat nor a division by a routing weight.
    const MlpBwdEpiLayout L = mlp_bwd_epi_layout(mode, es, (size_t)Tk, d_model, d_expert, d_h);
    char *base = (char *)ws;
    void *dYu = base + L.dybar_u, *second = base + L.second, *dH = base + L.dh, *dHpre = base + L.dhpre;
    float *dp_part = (float *)(base + L.dp_part);
    float *tail_ws = (float *)(base + L.total - S2S_TAIL_WS_BYTES);
    // The W2^T product gathers the rows of dY itself (Alg. 1's scattered input, fan-out k), and groupXTY those of X, and of dY when the
    // weights go into Hw; otherwise it reads a routing-weighted sorted copy of dY.  Where groupXTY cannot gather (sources past 32-bit
    // offsets) or an output lies over X or dY, sorted copies stand in.
    const size_t x_bytes = (size_t)T * d_model * es, w1_bytes = (size_t)r->E * d_model * d_h * es, w2_bytes = (size_t)r->E * d_expert * d_model * es;
    const bool apart = !overlap(dW1, w1_bytes, X, x_bytes) && !overlap(dW2, w2_bytes, X, x_bytes) && !overlap(dW1, w1_bytes, dY, x_bytes) &&
                       !overlap(dW2, w2_bytes, dY, x_bytes) && !overlap(dgates, (size_t)Tk * sizeof(float), dY, x_bytes);
    const RowMap tokens{r->sorted_scattered_idxs, k};
    DWArgs w1{X, dHpre, dW1, r->expert_offsets, r->E, Tk, d_model, d_h};
    DWArgs w2{saved_H, second, dW2, r->expert_offsets, r->E, Tk, d_expert, d_model};
    w1.a_map = tokens;
    const bool rows_x = apart && dw_reads_rows(ctx, w1);
    // The weighted hidden rows Hw take the place of a weighted copy of dY where they are no wider: the layout has them beside the plain
    // copy of dY (mode 2), or they lie in the copy's own array when groupXTY gathers dY (mode 1).
    // Mode 1, 8192 tokens on 64 experts, k = 8, 2048 -> 2 x 512: the product that writes Hw takes 233 us, without it 232, and the copy
    // of dY was 50 with 5 for the inverse of the order indices; the training step 1545 -> 1481.  The error of dW2 against 64 bits, with
    // p dY / p H rounded, five layers of 264 to 2048: 2.348e-3 / 2.348e-3 (k = 1), 2.863 to 2.875 / 2.868 to 2.874.
    w2.B = dY;
    w2.b_map = tokens;
    const bool rows_y = d_expert <= d_model && apart && dw_reads_rows(ctx, w2);
    const bool hw = L.use_hw || rows_y;
    if (hw) w2.A = second;
    if (!rows_y) {
      w2.B = L.use_hw ? dYu : second;
      w2.b_map = RowMap{nullptr, 1};
    }
    int32_t *inv_y = (int32_t *)dp_part, *inv_x = k > 1 ? (int32_t *)(base + L.inv_x) : nullptr;
    // (spread: see the line in plinear_bwd; X's copy has its inverse at no cost)
    const bool spread_y = k > 1 && (size_t)Tk * d_model >= SPREAD_MIN_ELEMENTS;
    auto sorted_copy = [&](const void *rows, const int32_t *inv, const float *weights, void *out) {
      return inv ? launch_spread(s, rows, inv, k, weights, out, Tk, d_model)
                    : launch_group(s, dtype, rows, r->sorted_scattered_idxs, k, weights, out, Tk, d_model);
    };
    if (!rows_y) {
      if (spread_y) rc = launch_invert(s, r->sorted_scattered_idxs, inv_y, Tk);
      if (rc == SMOE_OK) rc = sorted_copy(dY, spread_y ? inv_y : nullptr, L.use_hw ? nullptr : gates, L.use_hw ? dYu : second);
      if (rc != SMOE_OK) return rc;
    }
    S2SArgs x2 = make_s2s(dY, W2, mode == 1 ? dHpre : dH, r, d_expert, d_model, true, false, k, true);
    if (mode == 1) {
      x2.Hpre_in = saved_Hpre;           // dHpre = sigma'(Hpre) p (dYu W2^T) straight from the accumulators
    }
    if (mode == 2 || hw) x2.H_in = saved_H;   // mode 2: dH = p (dYu W2^T); Hw = p H
    x2.Hw_out = hw ? second : nullptr;
    x2.row_scale = gates;
    x2.dp_part = dp_part;
    set_launch(ctx, x2);
    rc = launch_s2s_stream(s, x2);
    if (rc != SMOE_OK) return rc;
    rc = launch_dp_reduce(s, dp_part, L.part_ld, r->sorted_scattered_idxs, dgates, rows_x ? nullptr : inv_x, Tk);
    if (rc != SMOE_OK) return rc;
    if (mode == 2) {
      rc = launch_act_bwd(s, act, saved_Hpre, dH, dHpre, Tk, d_expert);
      if (rc != SMOE_OK) return rc;
    }
    w2.split_ws = tail_ws;
    void *Xbar = L.use_hw ? dYu : second;                // dead after dW2: its array holds Xbar where that is made, then dXbar
    // Both weight gradients in one launch where that saves a round of tiles.  A sorted copy of X would take the room of the partial
    // tiles, which nothing needs until the last product.
    DWArgs both = w2;
    both.A3 = rows_x ? X : tail_ws;
    both.a3_map = rows_x ? tokens : RowMap{nullptr, 1};
    both.order = r->sorted_scattered_idxs;
    both.B3 = dHpre;
    both.dW3 = dW1;
    both.M3 = d_model;
    both.N3 = d_h;
    both.grid = ctx->stream_grid;
    if ((rows_x || (size_t)Tk * d_model * es <= S2S_TAIL_WS_BYTES) && !overlap(dW1, w1_bytes, saved_H, (size_t)Tk * d_expert * es) &&
        dw_stream_supported(both) && dw_stream_two_pay(both)) {
      if (!rows_x) rc = sorted_copy(X, inv_x, nullptr, tail_ws);
      if (rc == SMOE_OK) rc = launch_dw_stream(s, both);
      if (rc != SMOE_OK) return rc;
    } else {
      rc = run_dw(ctx, s, dtype, w2);
      if (rc != SMOE_OK) return rc;
      if (!rows_x) {
        rc = sorted_copy(X, inv_x, nullptr, Xbar);
        if (rc != SMOE_OK) return rc;
        w1.A = Xbar;
        w1.a_map = RowMap{nullptr, 1};
      }
      w1.split_ws = tail_ws;
      rc = run_dw(ctx, s, dtype, w1);
      if (rc != SMOE_OK) return rc;
    }
    S2SArgs x1 = make_s2s(dHpre, W1, k == 1 ? dX : Xbar, r, d_model, d_h, true, true, 1, false);
    x1.tail_ws = tail_ws;
    rc = run_s2s(ctx, s, dtype, x1);
    if (rc != SMOE_OK || k == 1) return rc;
    return launch_combine(s, dtype, Xbar, nullptr, dX, T, k, d_model);
  }
  char *p = (char *)ws;
  void *dYbar = p;                 p += align256((size_t)Tk * d_model * es);
  void *dH = p;                    p += align256((size_t)Tk * d_expert * es);
  void *dHpre = p;
  float *tail_ws = (float *)((char *)ws + need - S2S_TAIL_WS_BYTES);   // partial tiles of a split last round
  void *Xbar = dYbar;  // dYbar is dead once dH and dW2 are done; its array then holds Xbar, then dXbar

  // ---- second ParallelLinear (grouped in, scattered weighted out)
  if (dtype == SMOE_F32) {
    // The fp32 kernels gather and weight rows where they read them and apply the activation's derivative in the epilogue.
    const RowMap tokens{r->sorted_scattered_idxs, k};
    DWArgs w2{saved_H, dY, dW2, r->expert_offsets, r->E, Tk, d_expert, d_model};
    w2.b_map = tokens;
    w2.gates = gates;
    S2SArgs x2 = make_s2s(dY, W2, dHpre, r, d_expert, d_model, true, false, k, true);
    x2.Hpre_in = saved_Hpre;
    x2.act = act;
    x2.gates = gates;
    x2.slots = r->sorted_scattered_idxs;
    const RowDots d{dY, saved_Yhat, dgates, Tk, k, d_model};                              // dp = bmm(dY, Yhat)
    const size_t w2_bytes = (size_t)r->E * d_expert * d_model * 4, row_bytes = (size_t)Tk * 4;
    rc = run_f32_backward(s, x2, w2, d, overlap(dW2, w2_bytes, saved_Yhat, row_bytes * d_model) || overlap(dW2, w2_bytes, dgates, row_bytes));
    if (rc != SMOE_OK) return rc;
    DWArgs w1{X, dHpre, dW1, r->expert_offsets, r->E, Tk, d_model, d_h};
    w1.a_map = tokens;
    void *dst = k == 1 ? dX : Xbar;
    rc = run_f32_backward(s, make_s2s(dHpre, W1, dst, r, d_model, d_h, true, true, 1, false), w1, RowDots{},
                          overlap(dst, row_bytes * d_model, X, (size_t)T * d_model * 4) ||
                              overlap(dst, row_bytes * d_model, dW1, (size_t)r->E * d_model * d_h * 4));
    if (rc != SMOE_OK || k == 1) return rc;
    return launch_combine(s, dtype, Xbar, nullptr, dX, T, k, d_model);
  }
  rc = launch_rowdot(s, dtype, dY, saved_Yhat, dgates, Tk, k, d_model);                 // dp = bmm(dY, Yhat)
  if (rc != SMOE_OK) return rc;
  rc = launch_group(s, dtype, dY, r->sorted_scattered_idxs, k, gates, dYbar, Tk, d_model);  // weight and group
  if (rc != SMOE_OK) return rc;
  DWArgs w2{saved_H, dYbar, dW2, r->expert_offsets, r->E, Tk, d_expert, d_model};
  w2.split_ws = tail_ws;
  rc = run_dw(ctx, s, dtype, w2);                                                      // groupXTY
  if (rc != SMOE_OK) return rc;
  S2SArgs x2 = make_s2s(dYbar, W2, dH, r, d_expert, d_model, true, true, 1, true);      // dH = dYbar W2^T
  x2.tail_ws = tail_ws;
  rc = run_s2s(ctx, s, dtype, x2);
  if (rc != SMOE_OK) return rc;
  // ---- activation
  rc = launch_act_bwd(s, act, saved_Hpre, dH, dHpre, Tk, d_expert);
  if (rc != SMOE_OK) return rc;
  // ---- first ParallelLinear (scattered in with fan-out k, grouped out): its one `group`
  rc = launch_group(s, dtype, X, r->sorted_scattered_idxs, k, nullptr, Xbar, Tk, d_model);
  if (rc != SMOE_OK) return rc;
  DWArgs w1{Xbar, dHpre, dW1, r->expert_offsets, r->E, Tk, d_model, d_h};
  w1.split_ws = tail_ws;
  rc = run_dw(ctx, s, dtype, w1);
  if (rc != SMOE_OK) return rc;
  if (k == 1) {  // slot id == token id: scatter straight into dX
    S2SArgs x1 = make_s2s(dHpre, W1, dX, r, d_model, d_h, true, true, 1, false);
    x1.tail_ws = tail_ws;
    return run_s2s(ctx, s, dtype, x1);
  }
  S2SArgs x1 = make_s2s(dHpre, W1, Xbar, r, d_model, d_h, true, true, 1, false);        // grouped -> scattered dXbar
  x1.tail_ws = tail_ws;
  rc = run_s2s(ctx, s, dtype, x1);
  if (rc != SMOE_OK) return rc;
  return launch_combine(s, dtype, Xbar, nullptr, dX, T, k, d_model);                    // sum the k slots
}

// ------------------------------------------------------------------------------ Alg. 4
namespace {
struct MomhaSizes {
  size_t kv, q, lse, yhat, x;   // bytes, each rounded up to 256
};
MomhaSizes momha_sizes(int B, int T, int k, int d_model, int h_expert, int d_head) {
  size_t N = (size_t)B * T, Tk = N * k, d_out = (size_t)h_expert * d_head;
  return MomhaSizes{align256(N * d_out * 2), align256(Tk * d_out * 2), align256(Tk * h_expert * sizeof(float)),
                    align256(Tk * d_model * 2), align256(N * d_model * 2)};
}
int momha_args_ok(smoe_ctx *ctx, smoe_dtype dtype, int B, int T, int d_model, int h_expert, int d_head,
                  const smoe_routing *r, int k) {
  if (!ctx || !routing_ok(r) || d_model < 1 || k < 1) return SMOE_ERR_INVALID_ARG;
  int rc = attention_args_ok(dtype, B, T, k, h_expert, d_head);
  if (rc != SMOE_OK) return rc;
  if ((long long)B * T * k != r->Tk) return SMOE_ERR_INVALID_ARG;
  if (!width_ok(dtype, d_model)) return SMOE_ERR_UNSUPPORTED;
  return SMOE_OK;
}
// a dense product A [n, d_in] x W (or W^T) run through the grouped kernels as one expert
S2SArgs dense_s2s(const void *A, const void *W, void *C, const int32_t *offsets, int n, int d_in, int d_out, bool trans_w) {
  smoe_routing r{nullptr, nullptr, offsets, n, 1};
  return make_s2s(A, W, C, &r, d_in, d_out, trans_w, true, 1, true);
}
// Two dense products (two weight gradients) of the same sizes, in one launch where the persistent kernels take them: alone
// each fills half of the chip at the widths of a key or value projection (8192 rows, 2048 -> 512: 2 x 41 us, paired 43; the
// weight gradients 2 x 57 us, paired 58).
// The persistent kernels know two segments of equal length without being given their offsets; the others read them from `off`.
int run_s2s_pair(smoe_ctx *ctx, hipStream_t s, const S2SArgs &a, const S2SArgs &b, int32_t *off) {
  S2SArgs p = a;
  p.E = 2;
  p.Tk = 2 * a.Tk;
  p.offsets = nullptr;
  p.A2 = (const void *)((uintptr_t)b.A - (uintptr_t)a.Tk * a.K * 2);
  p.W2 = (const void *)((uintptr_t)b.W - (uintptr_t)a.w_stride * 2);
  p.C2 = (void *)((uintptr_t)b.C - (uintptr_t)a.Tk * a.N * 2);
  set_launch(ctx, p);
  if (ctx->kernel_mode == 0 && a.Tk < (1 << 30) && !s2s_decode_supported(a) && s2s_stream_supported(p)) return launch_s2s_stream(s, p);
  int rc = launch_dense_offsets(s, off, a.Tk);
  if (rc == SMOE_OK) rc = run_s2s(ctx, s, SMOE_BF16, a);
  return rc != SMOE_OK ? rc : run_s2s(ctx, s, SMOE_BF16, b);
}
int run_dw_pair(smoe_ctx *ctx, hipStream_t s, const DWArgs &a, const DWArgs &b, int32_t *off) {
  DWArgs p = a;
  p.E = 2;
  p.Tk = 2 * a.Tk;
  p.offsets = nullptr;
  p.A2 = (const void *)((uintptr_t)b.A - (uintptr_t)a.Tk * a.M * 2);
  p.B2 = (const void *)((uintptr_t)b.B - (uintptr_t)a.Tk * a.N * 2);
  p.dW2 = (void *)((uintptr_t)b.dW - (uintptr_t)a.M * a.N * 2);
  p.grid = ctx->stream_grid;
  if (ctx->kernel_mode == 0 && a.Tk < (1 << 30) && dw_stream_supported(p)) return launch_dw_stream(s, p);
  int rc = launch_dense_offsets(s, off, a.Tk);
  if (rc == SMOE_OK) rc = run_dw(ctx, s, SMOE_BF16, a);
  return rc != SMOE_OK ? rc : run_dw(ctx, s, SMOE_BF16, b);
}
}  // namespace

size_t smoe_momha_fwd_workspace_bytes(int B, int T, int k, int d_model, int h_expert, int d_head, int training) {
  if (B < 1 || T < 1 || k < 1 || d_model < 1 || h_expert < 1 || d_head < 1) return 0;
  MomhaSizes z = momha_sizes(B, T, k, d_model, h_expert, d_head);
  return 256 + S2S_TAIL_WS_BYTES + (training ? 0 : 2 * z.kv + 2 * z.q + z.lse + z.yhat);
}

int smoe_momha_fwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *X, int B, int T, int d_model,
                   int h_expert, int d_head, const void *W_K, const void *W_V, const void *W_Q, const void *W_O,
                   const smoe_routing *r, int k, const float *gates, void *O, void *saved_K, void *saved_V,
                   void *saved_Q, void *saved_Ohat, float *saved_LSE, void *saved_Yhat, void *ws, size_t ws_bytes) {
  int rc = momha_args_ok(ctx, dtype, B, T, d_model, h_expert, d_head, r, k);
  if (rc != SMOE_OK) return rc;
  if (!X || !W_K || !W_V || !W_Q || !W_O || !gates || !O) return SMOE_ERR_INVALID_ARG;
  const int n_saved = !!saved_K + !!saved_V + !!saved_Q + !!saved_Ohat + !!saved_LSE + !!saved_Yhat;
  if (n_saved != 0 && n_saved != 6) return SMOE_ERR_INVALID_ARG;
  size_t need = smoe_momha_fwd_workspace_bytes(B, T, k, d_model, h_expert, d_head, n_saved == 6);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return SMOE_ERR_WORKSPACE;
  const int N = B * T, Tk = r->Tk, d_out = h_expert * d_head;
  MomhaSizes z = momha_sizes(B, T, k, d_model, h_expert, d_head);
  char *p = (char *)ws;
  int32_t *dense_off = (int32_t *)p;  p += 256;
  float *tail_ws = (float *)p;  p += S2S_TAIL_WS_BYTES;
  if (n_saved == 0) {
    saved_K = p;  p += z.kv;
    saved_V = p;  p += z.kv;
    saved_Q = p;  p += z.q;
    saved_Ohat = p;  p += z.q;
    saved_LSE = (float *)p;  p += z.lse;
    saved_Yhat = p;
  }
  hipStream_t s = (hipStream_t)stream;
  // V = X W_V, K = X W_K
  auto product = [&](S2SArgs a) { a.tail_ws = tail_ws; return run_s2s(ctx, s, dtype, a); };
  S2SArgs pv = dense_s2s(X, W_V, saved_V, dense_off, N, d_model, d_out, false);
  S2SArgs pk = dense_s2s(X, W_K, saved_K, dense_off, N, d_model, d_out, false);
  pv.tail_ws = pk.tail_ws = tail_ws;
  rc = run_s2s_pair(ctx, s, pv, pk, dense_off);
  if (rc != SMOE_OK) return rc;
  // Q = ParallelLinear(X, W_Q, o, no p, scattered -> scattered)
  rc = product(make_s2s(X, W_Q, saved_Q, r, d_model, d_out, false, false, k, false));
  if (rc != SMOE_OK) return rc;
  // Ohat = Attention(Q, K, V)
  rc = launch_attn_fwd(s, saved_Q, saved_K, saved_V, saved_Ohat, saved_LSE, B, T, k, h_expert);
  if (rc != SMOE_OK) return rc;
  // O = ParallelLinear(Ohat, W_O, o, p, scattered -> scattered)
  rc = product(make_s2s(saved_Ohat, W_O, saved_Yhat, r, d_out, d_model, false, false, 1, false));
  if (rc != SMOE_OK) return rc;
  return launch_combine(s, dtype, saved_Yhat, gates, O, N, k, d_model);
}

// Does forming dp in the epilogue of the output projection's input-gradient product pay?  It saves passes over rows of [Tk, d_model],
// and its epilogue gains on them only where these are long enough (16 Mi elements).  Backward pass of the layer, 8 experts, sequences of
// 512, in us, with it / without, rows x d_model, heads, k:
//   both lines met:  32768 x 512, 2, 4: 290 / 305; 16384 x 1024, 4, 4: 346 / 359; 65536 x 256, 4, 8: 534 / 536; 65536 x 2048, 2, 8:
//                    666 / 798; 32768 x 2048, 4, 4: 671 / 720; 32768 x 1024, 8, 2: 801 / 800; 16384 x 1024, 8, 4: 482 / 482;
//   8 Mi elements:   128 tiles 32768 x 256, 2, 4: 263 / 266, 16384 x 512, 4, 8: 293 / 292, 8192 x 1024, 8, 8: 282 / 282; 256 tiles
//                    16384 x 512, 8, 4: 426 / 414, 32768 x 256, 4, 2: 395 / 387; 512 tiles 32768 x 256, 8, 4: 559 / 539;
//   4 Mi:            256 tiles 16384 x 256, 8, 4: 377 / 371, 512 tiles 32768 x 128, 8, 2: 518 / 493.
// The line at 128 tiles (half a round of 256 x 256) was drawn when the product ran on such tiles alone and lost under it.  On the smaller
// ones it wins there: 64 tiles 16384 x 1024, 2, 8: 272 / 283; 8192 x 2048, 4, 8: 258 / 269; 16384 x 2048, 1, 8: 306 / 334.  It stays for
// dgates' sake: fp32, and rounded otherwise on the other route, by 1e-3.
static bool output_projection_in_epilogue(const smoe_ctx *ctx, int Tk, int d_model, int d_out) {
  if (ctx->tile_shape) return ctx->tile_shape == 2;   // tiles of one shape only, for the tests
  return (size_t)Tk * d_model >= ((size_t)16 << 20) && (long long)ceil_div(Tk, 256) * ceil_div(d_out, 256) * 2 >= ctx->stream_grid;
}

size_t smoe_momha_bwd_workspace_bytes(int B, int T, int k, int d_model, int h_expert, int d_head) {
  if (B < 1 || T < 1 || k < 1 || d_model < 1 || h_expert < 1 || d_head < 1) return 0;
  MomhaSizes z = momha_sizes(B, T, k, d_model, h_expert, d_head);
  // dense offsets, dOhat, dQ, dK, dV, three partial dX, delta, and the ParallelLinear backward scratch
  // (a grouped [Tk, d_model] and a grouped [Tk, d_out] array, used by both projections in turn)
  return 256 + 2 * z.q + 2 * z.kv + 3 * z.x + smoe_attention_bwd_workspace_bytes(B, T, k, h_expert) + z.yhat + z.q +
         S2S_TAIL_WS_BYTES;
}

int smoe_momha_bwd(smoe_ctx *ctx, void *stream, smoe_dtype dtype, const void *dO, const void *X, int B, int T,
                   int d_model, int h_expert, int d_head, const void *W_K, const void *W_V, const void *W_Q,
                   const void *W_O, const smoe_routing *r, int k, const float *gates, const void *saved_K,
                   const void *saved_V, const void *saved_Q, const void *saved_Ohat, const float *saved_LSE,
                   const void *saved_Yhat, void *dX, void *dW_K, void *dW_V, void *dW_Q, void *dW_O, float *dgates,
                   void *ws, size_t ws_bytes) {
  int rc = momha_args_ok(ctx, dtype, B, T, d_model, h_expert, d_head, r, k);
  if (rc != SMOE_OK) return rc;
  if (!dO || !X || !W_K || !W_V || !W_Q || !W_O || !gates || !saved_K || !saved_V || !saved_Q || !saved_Ohat ||
      !saved_LSE || !saved_Yhat || !dX || !dW_K || !dW_V || !dW_Q || !dW_O || !dgates)
    return SMOE_ERR_INVALID_ARG;
  size_t need = smoe_momha_bwd_workspace_bytes(B, T, k, d_model, h_expert, d_head);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return SMOE_ERR_WORKSPACE;
  // what the two ParallelLinears' backward passes ask of their operands, asked before anything is enqueued
  if (!aligned16(dO) || !aligned16(X) || !aligned16(saved_Ohat) || !aligned16(W_Q) || !aligned16(W_O) || !aligned16(dW_Q) || !aligned16(dW_O))
    return SMOE_ERR_UNSUPPORTED;
  const int N = B * T, Tk = r->Tk, d_out = h_expert * d_head;
  MomhaSizes z = momha_sizes(B, T, k, d_model, h_expert, d_head);
  char *p = (char *)ws;
  int32_t *dense_off = (int32_t *)p;  p += 256;
  void *dOhat = p;  p += z.q;
  void *dQ = p;     p += z.q;
  void *dK = p;     p += z.kv;
  void *dV = p;     p += z.kv;
  void *dXq = p;    p += z.x;
  void *dXk = p;    p += z.x;
  void *dXv = p;    p += z.x;
  void *attn_ws = p;  p += smoe_attention_bwd_workspace_bytes(B, T, k, h_expert);
  void *sub = p;
  const size_t sub_bytes = z.yhat + z.q + S2S_TAIL_WS_BYTES;
  float *tail_ws = (float *)((char *)sub + z.yhat + z.q);   // where the ParallelLinear backward puts its own, too
  hipStream_t s = (hipStream_t)stream;
  const bool in_sum = k > 1 && aligned16(dX);   // dXk and dXv are added where the k slots of dX are summed, whose kernel writes 16-byte lines
  // the array of dX's third part is free then: it holds the inverse of the order indices
  int32_t *inv = in_sum && (size_t)Tk * sizeof(int32_t) <= z.x ? (int32_t *)dXq : nullptr;
  // Output projection (Alg. 2 with p, scattered in with fan-out 1, scattered out): dOhat, dW_O, dp.  Where the persistent kernels take
  // the product, its epilogue reads the saved Ohat, leaves <dO W_O^T, Ohat> in slabs, which add up to dp, and writes the weighted,
  // sorted rows of Ohat that groupXTY needs.  No pass over Yhat, no `group` of Ohat (34 + 14 us at 8192 tokens, k = 4, 4 heads, 2048
  // wide).  The attention's delta = <dOhat, Ohat> is not taken from there: it has to go with dOhat as it is stored.
  const int part_ld = 2 * ceil_div(d_out, 256);
  float *dp_part = tail_ws;
  void *dYu = sub, *Ow = (char *)sub + z.yhat;
  S2SArgs xo = make_s2s(dO, W_O, dOhat, r, d_out, d_model, true, false, k, false);
  xo.H_in = saved_Ohat;
  xo.Hw_out = Ow;
  xo.row_scale = gates;
  xo.dp_part = dp_part;
  set_launch(ctx, xo);
  const bool in_epilogue = inv && ctx->kernel_mode == 0 && s2s_stream_dp_supported(xo) && output_projection_in_epilogue(ctx, Tk, d_model, d_out) &&
                           (size_t)Tk * part_ld * sizeof(float) <= S2S_TAIL_WS_BYTES;
  if (in_epilogue) {
    rc = launch_invert(s, r->sorted_scattered_idxs, inv, Tk);
    if (rc != SMOE_OK) return rc;
    rc = launch_s2s_stream(s, xo);
    if (rc != SMOE_OK) return rc;
    rc = launch_dp_reduce(s, dp_part, part_ld, r->sorted_scattered_idxs, dgates, nullptr, Tk);
    if (rc != SMOE_OK) return rc;
    DWArgs wo{Ow, dO, dW_O, r->expert_offsets, r->E, Tk, d_out, d_model};
    wo.b_map = RowMap{r->sorted_scattered_idxs, k};
    if (overlap(dW_O, (size_t)r->E * d_out * d_model * 2, dO, (size_t)N * d_model * 2) || !dw_reads_rows(ctx, wo)) {
      rc = launch_spread(s, dO, inv, k, nullptr, dYu, Tk, d_model);
      if (rc != SMOE_OK) return rc;
      wo.B = dYu;
      wo.b_map = RowMap{nullptr, 1};
    }
    wo.split_ws = tail_ws;
    rc = run_dw(ctx, s, dtype, wo);
  } else {
    rc = smoe_plinear_bwd(ctx, stream, dtype, dO, saved_Ohat, Tk, d_out, W_O, d_model, saved_Yhat, r, 1, gates, k, 0, 0,
                          dOhat, dW_O, dgates, sub, sub_bytes);
    if (rc == SMOE_OK && inv) rc = launch_invert(s, r->sorted_scattered_idxs, inv, Tk);
  }
  if (rc != SMOE_OK) return rc;
  // with the inverse at hand dQ is written in expert-sorted order, as the query projection's gradients read it
  rc = launch_attn_bwd(s, saved_Q, saved_K, saved_V, saved_Ohat, dOhat, saved_LSE, attn_ws, dQ, dK, dV, B, T, k, h_expert, true, inv);
  if (rc != SMOE_OK) return rc;
  // dense key / value projections
  DWArgs wk{X, dK, dW_K, dense_off, 1, N, d_model, d_out}, wv{X, dV, dW_V, dense_off, 1, N, d_model, d_out};
  wk.split_ws = wv.split_ws = (float *)((char *)sub + z.yhat + z.q);
  rc = run_dw_pair(ctx, s, wk, wv, dense_off);
  if (rc != SMOE_OK) return rc;
  S2SArgs xk = dense_s2s(dK, W_K, dXk, dense_off, N, d_model, d_out, true);
  S2SArgs xv = dense_s2s(dV, W_V, dXv, dense_off, N, d_model, d_out, true);
  xk.tail_ws = xv.tail_ws = tail_ws;
  rc = run_s2s_pair(ctx, s, xk, xv, dense_off);
  if (rc != SMOE_OK) return rc;
  // query projection (Alg. 2 without p, scattered in with fan-out k, scattered out): dW_Q, and dX = its part + dXk + dXv
  rc = plinear_bwd(ctx, stream, dtype, dQ, X, N, d_model, W_Q, d_out, nullptr, r, k, nullptr, 0, 0, inv ? 1 : 0, in_sum ? dX : dXq, dW_Q, nullptr, sub,
                   sub_bytes, in_sum ? dXk : nullptr, in_sum ? dXv : nullptr, inv);
  if (rc != SMOE_OK || in_sum) return rc;
  return launch_add3(s, dXq, dXk, dXv, dX, (size_t)N * d_model);
}

}  // extern "C"
