// Grouped GEMMs in fp32 arithmetic on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums), for fp32 tensors
// and for the bf16 shapes the bf16 matrix-core kernels do not take.  Same operations as those: scatter2scatter (Sec. 3.2)
// with W or W^T, and groupXTY (Sec. 3.2.1).
//
// The fp32 layers are small, so what bounds them is latency: launches, and in a launch the chain offsets -> order index ->
// operand row -> result.  Hence: rows are gathered (and weighted) where they are read instead of by a `group` launch, the
// activation and its derivative sit in the epilogues instead of launches of their own, the tile search runs across the
// lanes of a wavefront, row addresses are worked out once, each 32-deep contraction step is loaded into registers while the one before
// is multiplied, and the parts of a backward pass that wait for nothing but their inputs are one launch (f32_backward_kernel).
// In us, and before the backward passes were one launch a layer: 256 tokens, 64 -> 128 -> 64, 4 experts: forward 16, backward 19 (36);
// 1024 tokens, 256 -> 2 x 896 -> 256, 8 experts, k = 2: 61 and 97 (131); 4096 tokens, 256 -> 512 -> 256: 68 and 123 (160); 16384 tokens,
// 1024 -> 4096 -> 1024: 5540 and 10640 (12240), 99 and 103 TFLOP/s of the card's 157 in fp32.
// Steps requested two ahead into a second set of registers and LDS tiles leave 4 wavefronts a SIMD of 6 to 8 and were slower by 2 to 8 %
// in the forward products and by up to 15 % in the backward launches (65 and 112 us for the 1024 tokens); the longest weight
// gradients of few tiles gained 2 to 3 % (32768 tokens, 128 -> 256 -> 128, 16 experts: 356 us, 365 so).
#include "mfma_common.h"

namespace {
constexpr int PT = 64;        // tile edge (rows and columns); four wavefronts of 32 x 32
constexpr int PK = 32;        // contraction step
constexpr int KROW = PK + 4;  // floats per row of a [row][k] operand tile: the pad keeps its 16-byte reads conflict free
constexpr int NROW = PT + 4;  // floats per row of a [k][column] operand tile

template <typename T> struct Vec16 { static constexpr int N = 16 / sizeof(T); T v[N]; } __attribute__((aligned(16)));

// An operand tile on its way through registers: 64 x 32 elements, 16-byte vectors dealt to the 256 threads.
template <typename T> struct TileRegs {
  static constexpr int V = 16 / sizeof(T), U = PT * PK / V / 256;
  Vec16<T> r[U];
};
// [row][k] tile (contraction contiguous): vector u of a thread belongs to row(u) and starts at k(u)
template <typename T> __device__ __forceinline__ int kc_row(int u) { constexpr int V = 16 / sizeof(T); return (threadIdx.x + 256 * u) / (PK / V); }
template <typename T> __device__ __forceinline__ int kc_k(int u) { constexpr int V = 16 / sizeof(T); return (threadIdx.x + 256 * u) % (PK / V) * V; }
// [k][column] tile (columns contiguous)
template <typename T> __device__ __forceinline__ int cc_k(int u) { constexpr int V = 16 / sizeof(T); return (threadIdx.x + 256 * u) / (PT / V); }
template <typename T> __device__ __forceinline__ int cc_col(int u) { constexpr int V = 16 / sizeof(T); return (threadIdx.x + 256 * u) % (PT / V) * V; }

template <typename T> __device__ __forceinline__ Vec16<T> load_or_zero(const T *p, bool ok) {
  Vec16<T> v{};
  if (ok) v = *reinterpret_cast<const Vec16<T> *>(p);
  return v;
}
template <typename T> __device__ __forceinline__ void put_floats(float *dst, const Vec16<T> &v, float scale) {
#pragma unroll
  for (int i = 0; i < Vec16<T>::N; i += 4)
    *reinterpret_cast<float4 *>(dst + i) = make_float4(scale * to_f32<T>(v.v[i]), scale * to_f32<T>(v.v[i + 1]), scale * to_f32<T>(v.v[i + 2]),
                                                       scale * to_f32<T>(v.v[i + 3]));
}
template <typename T> __device__ __forceinline__ void store4(T *p, float a, float b, float c, float d) {
  p[0] = from_f32<T>(a); p[1] = from_f32<T>(b); p[2] = from_f32<T>(c); p[3] = from_f32<T>(d);
}
template <> __device__ __forceinline__ void store4<float>(float *p, float a, float b, float c, float d) {
  *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, d);
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t *p, float a, float b, float c, float d) {
  bf16x4 v;
  v[0] = (bf16_t)a; v[1] = (bf16_t)b; v[2] = (bf16_t)c; v[3] = (bf16_t)d;
  *reinterpret_cast<bf16x4 *>(p) = v;
}
// One step: a lane of half h takes contraction elements 8 g + 4 h + j; the matrix instruction j contracts the pair (h = 0, 1).
// KC operands come four at a time (one 16-byte read), CC operands one by one.
__device__ __forceinline__ void frag_kc(float (&f)[4], const float *tile, int base, int g, int lane) {
  const float4 v = *reinterpret_cast<const float4 *>(tile + (base + (lane & 31)) * KROW + 8 * g + 4 * (lane >> 5));
  f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
__device__ __forceinline__ void frag_cc(float (&f)[4], const float *tile, int base, int g, int lane) {
#pragma unroll
  for (int j = 0; j < 4; ++j) f[j] = tile[(8 * g + 4 * (lane >> 5) + j) * NROW + base + (lane & 31)];
}
template <bool A_KC, bool B_KC>
__device__ __forceinline__ void multiply_step(const float *As, const float *Bs, int wm, int wn, int lane, f32x16 &acc) {
#pragma unroll
  for (int g = 0; g < PK / 8; ++g) {
    float fa[4], fb[4];
    if (A_KC) frag_kc(fa, As, wm * 32, g, lane); else frag_cc(fa, As, wm * 32, g, lane);
    if (B_KC) frag_kc(fb, Bs, wn * 32, g, lane); else frag_cc(fb, Bs, wn * 32, g, lane);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j], fa[j], acc, 0, 0, 0);
  }
}

// Epilogue: ACT_FWD  C (when given) = product, H = act(product); for SwiGLU a tile holds 32 gate columns and the 32 up
//                    columns pairing with them.
//           ACT_BWD  C = act'(Hpre) * product (SwiGLU: both halves).
// Rows of the product are scaled by the routing weight of their slot when a.gates is given.
enum { EPI_NONE = 0, EPI_ACT_FWD = 1, EPI_ACT_BWD = 2 };
constexpr int TILE_FLOATS = PT * KROW > PK * NROW ? PT * KROW : PK * NROW;
struct PlainTiles {
  float a[TILE_FLOATS], b[TILE_FLOATS];
};
template <typename T, bool TRANS_W, int EPI>
__device__ __forceinline__ void s2s_plain_tile(const S2SArgs &a, int mt, int nt, PlainTiles &tiles) {
  constexpr int U = TileRegs<T>::U;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
  int e, row0, row_end;
  if (!locate_rows<PT>(a.offsets, a.E, mt, lane, e, row0, row_end)) return;
  const bool swiglu = a.act == SMOE_ACT_SWIGLU, paired = EPI == EPI_ACT_FWD && swiglu;
  const int half_n = a.N / 2, n0 = nt * (paired ? 32 : PT);
  const T *W = (const T *)a.W + (size_t)e * a.w_stride;
  // column of the product that tile column c stands for
  auto column = [&](int c) { return !paired ? n0 + c : (c < 32 ? (n0 + c < half_n ? n0 + c : a.N) : (n0 + c - 32 < half_n ? half_n + n0 + c - 32 : a.N)); };

  const T *pa[U], *pb[U];
  bool oka[U], okb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = row0 + kc_row<T>(u);
    oka[u] = i < row_end;
    pa[u] = (const T *)a.A + (size_t)(oka[u] ? map_row(a.a_map, i) : 0) * a.K + kc_k<T>(u);
    if (TRANS_W) {
      const int n = n0 + kc_row<T>(u);
      okb[u] = n < a.N;
      pb[u] = W + (size_t)(okb[u] ? n : 0) * a.ldw + kc_k<T>(u);
    } else {
      const int n = column(cc_col<T>(u));
      okb[u] = n < a.N;
      pb[u] = W + (size_t)cc_k<T>(u) * a.ldw + (okb[u] ? n : 0);
    }
  }
  TileRegs<T> ra, rb;
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ra.r[u] = load_or_zero(pa[u] + k0, oka[u] && k0 + kc_k<T>(u) < a.K);
      rb.r[u] = TRANS_W ? load_or_zero(pb[u] + k0, okb[u] && k0 + kc_k<T>(u) < a.K)
                        : load_or_zero(pb[u] + (size_t)k0 * a.ldw, okb[u] && k0 + cc_k<T>(u) < a.K);
    }
  };
  fetch(0);
  // a lane holds row lane % 32 and the columns 8 g + 4 * (lane / 32) + 0..3 of its wavefront's 32 x 32 block
  const int i = row0 + wm * 32 + (lane & 31);
  const bool live = i < row_end;
  const size_t dst = live ? (size_t)map_row(a.c_map, i) : 0;
  const float scale = a.gates && live ? a.gates[a.slots[i]] : 1.0f;
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  for (int k0 = 0; k0 < a.K; k0 += PK) {
    if (k0) __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      put_floats<T>(tiles.a + kc_row<T>(u) * KROW + kc_k<T>(u), ra.r[u], 1.0f);
      if (TRANS_W) put_floats<T>(tiles.b + kc_row<T>(u) * KROW + kc_k<T>(u), rb.r[u], 1.0f);
      else put_floats<T>(tiles.b + cc_k<T>(u) * NROW + cc_col<T>(u), rb.r[u], 1.0f);
    }
    __syncthreads();
    if (k0 + PK < a.K) fetch(k0 + PK);
    multiply_step<true, TRANS_W>(tiles.a, tiles.b, wm, wn, lane, acc);
  }

  Vec16<float> pre[4], pre_up[4];          // EPI_ACT_BWD (fp32): the saved pre-activations of the lane's elements, all in flight at once
  if (EPI == EPI_ACT_BWD) {
    const float *h = (const float *)a.Hpre_in + (size_t)(live ? i : 0) * (swiglu ? 2 * a.N : a.N);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = column(wn * 32 + 8 * g + 4 * (lane >> 5));
      pre[g] = load_or_zero(h + n, live && n < a.N);
      pre_up[g] = load_or_zero(h + a.N + n, swiglu && live && n < a.N);
    }
  }
  float4 *exchange = reinterpret_cast<float4 *>(tiles.a);     // SwiGLU: the up columns cross over to the gate columns' wavefront
  if (paired) {
    __syncthreads();
    if (wn == 1)
#pragma unroll
      for (int g = 0; g < 4; ++g) exchange[(wm * 4 + g) * 64 + lane] = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    __syncthreads();
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = column(wn * 32 + 8 * g + 4 * (lane >> 5));
    if (!live || n >= a.N) continue;
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = scale * acc[4 * g + q];
    if (EPI == EPI_ACT_BWD) {
      const int d_h = swiglu ? 2 * a.N : a.N;
      T *out = (T *)a.C + dst * d_h + n;
      float x[4], y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float h = pre[g].v[q];
        if (swiglu) {
          const float u = pre_up[g].v[q], sg = sigmoid_f(h), silu = h * sg;
          x[q] = v[q] * u * (sg + silu * (1.0f - sg));
          y[q] = v[q] * silu;
        } else {
          x[q] = a.act == SMOE_ACT_GELU ? v[q] * gelu_grad_f(h) : v[q];
        }
      }
      store4<T>(out, x[0], x[1], x[2], x[3]);
      if (swiglu) store4<T>(out + a.N, y[0], y[1], y[2], y[3]);
      continue;
    }
    if (EPI == EPI_NONE || a.C) store4<T>((T *)a.C + dst * a.N + n, v[0], v[1], v[2], v[3]);
    if (EPI == EPI_ACT_FWD) {
      float h[4];
      if (swiglu) {
        if (wn == 1) continue;
        const float4 u = exchange[(wm * 4 + g) * 64 + lane];
        const float up[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = v[q] * sigmoid_f(v[q]) * up[q];
        store4<T>((T *)a.H + dst * half_n + n, h[0], h[1], h[2], h[3]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = a.act == SMOE_ACT_GELU ? gelu_f(v[q]) : v[q];
        store4<T>((T *)a.H + dst * a.N + n, h[0], h[1], h[2], h[3]);
      }
    }
  }
}

template <typename T, bool TRANS_W, int EPI>
__global__ void __launch_bounds__(256) s2s_plain_kernel(S2SArgs a) {
  __shared__ PlainTiles tiles;
  s2s_plain_tile<T, TRANS_W, EPI>(a, blockIdx.x, blockIdx.y, tiles);
}

// dW[e] = sum_i A[i, :]^T B[i, :] over the expert's rows; both operands may be gathered, B's rows weighted.
template <typename T> __device__ __forceinline__ void dw_plain_tile(const DWArgs &a, int nt, int mt, int e, PlainTiles &tiles) {
  constexpr int U = TileRegs<T>::U;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
  const int lo = a.offsets[e], hi = a.offsets[e + 1];
  const int m0 = mt * PT, n0 = nt * PT;
  TileRegs<T> ra, rb;
  float weight[U];
  // Order indices are fetched a step ahead of the rows they lead to, so that a step waits for one memory latency, not two.
  const int32_t *o = a.a_map.o ? a.a_map.o : a.b_map.o;   // both maps use the same order indices
  int slot[U];
  auto fetch_slots = [&](int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) slot[u] = o && i0 + cc_k<T>(u) < hi ? o[i0 + cc_k<T>(u)] : 0;
  };
  auto source = [&](const RowMap &map, int i, int u) { return (size_t)(map.o ? (map.fan > 1 ? slot[u] / map.fan : slot[u]) : i); };
  auto fetch = [&](int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + cc_k<T>(u), m = m0 + cc_col<T>(u), n = n0 + cc_col<T>(u);
      const bool ok = i < hi;
      weight[u] = a.gates && ok ? a.gates[slot[u]] : 1.0f;
      ra.r[u] = load_or_zero((const T *)a.A + (ok ? source(a.a_map, i, u) : 0) * a.M + (m < a.M ? m : 0), ok && m < a.M);
      rb.r[u] = load_or_zero((const T *)a.B + (ok ? source(a.b_map, i, u) : 0) * a.N + (n < a.N ? n : 0), ok && n < a.N);
    }
    fetch_slots(i0 + PK);
  };
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.f;
  fetch_slots(lo);
  fetch(lo);
  for (int i0 = lo; i0 < hi; i0 += PK) {
    if (i0 > lo) __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      put_floats<T>(tiles.a + cc_k<T>(u) * NROW + cc_col<T>(u), ra.r[u], 1.0f);
      put_floats<T>(tiles.b + cc_k<T>(u) * NROW + cc_col<T>(u), rb.r[u], weight[u]);
    }
    __syncthreads();
    if (i0 + PK < hi) fetch(i0 + PK);
    multiply_step<false, false>(tiles.a, tiles.b, wm, wn, lane, acc);
  }
  const int m = m0 + wm * 32 + (lane & 31);
  if (m >= a.M) return;
  T *dst = (T *)a.dW + ((size_t)e * a.M + m) * a.N;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = n0 + wn * 32 + 8 * g + 4 * (lane >> 5);
    if (n < a.N) store4<T>(dst + n, acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
  }
}

template <typename T> __global__ void __launch_bounds__(256) dw_plain_kernel(DWArgs a) {
  __shared__ PlainTiles tiles;
  dw_plain_tile<T>(a, blockIdx.x, blockIdx.y, blockIdx.z, tiles);
}

// What the backward pass of one fp32 ParallelLinear has to do, none of which waits for another part: the input-gradient product
// (EPI_ACT_BWD: with the activation's derivative), the weight gradient and the row dots of dp.  One launch instead of three: at
// these sizes a launch has 24 blocks or fewer for 256 compute units, and the gap to the next is 4 us (256 tokens, 64 -> 128 -> 64, 4
// experts: 2.9 + 9.2 + 9.4 us and two gaps became 9.5, 8.3 + 6.1 us and one gap 9.1).  The blocks with the longer walk go first (x_first:
// the contraction is longer than the average segment), else a short row of long walks ends the launch alone while the weight
// gradient's stores fill the memory queues (600 rows, 512 -> 2048, 8 experts: 65 us this way, 70 to 95 by where the arrays lie the
// other way, 83 in three launches).
template <int EPI> __global__ void __launch_bounds__(256) f32_backward_kernel(S2SArgs x, DWArgs w, RowDots d, int w_blocks, int x_blocks, bool x_first) {
  __shared__ PlainTiles tiles;
  int b = blockIdx.x;
  if (x_first && b < w_blocks + x_blocks) b = b < x_blocks ? b + w_blocks : b - x_blocks;
  if (b < w_blocks) {
    const int tn = (w.N + PT - 1) / PT, tm = (w.M + PT - 1) / PT;
    dw_plain_tile<float>(w, b % tn, b / tn % tm, b / tn / tm, tiles);
    return;
  }
  b -= w_blocks;
  if (b < x_blocks) {
    const int tn = (x.N + PT - 1) / PT;
    s2s_plain_tile<float, true, EPI>(x, b / tn, b % tn, tiles);
    return;
  }
  b -= x_blocks;
  const int s = b * 4 + (threadIdx.x >> 6);
  if (s < d.Tk) row_dot<float>(d, s, threadIdx.x & 63);
}

template <typename T, int EPI> void launch_s2s_plain_t(hipStream_t s, const S2SArgs &a) {
  const bool paired = EPI == EPI_ACT_FWD && a.act == SMOE_ACT_SWIGLU;
  const dim3 grid(ceil_div(a.Tk, PT) + a.E, paired ? ceil_div(a.N / 2, 32) : ceil_div(a.N, PT));
  if (a.trans_w) hipLaunchKernelGGL((s2s_plain_kernel<T, true, EPI>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((s2s_plain_kernel<T, false, EPI>), grid, dim3(256), 0, s, a);
}
}  // namespace

int launch_s2s_plain(hipStream_t s, smoe_dtype dt, const S2SArgs &a) {
  if (a.Tk == 0) return SMOE_OK;
  if (dt == SMOE_BF16) launch_s2s_plain_t<bf16_t, EPI_NONE>(s, a);
  else if (a.H) launch_s2s_plain_t<float, EPI_ACT_FWD>(s, a);
  else if (a.Hpre_in) launch_s2s_plain_t<float, EPI_ACT_BWD>(s, a);
  else launch_s2s_plain_t<float, EPI_NONE>(s, a);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

int launch_dw_plain(hipStream_t s, smoe_dtype dt, const DWArgs &a) {
  dim3 grid(ceil_div(a.N, PT), ceil_div(a.M, PT), a.E), block(256);
  if (dt == SMOE_BF16) hipLaunchKernelGGL((dw_plain_kernel<bf16_t>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((dw_plain_kernel<float>), grid, block, 0, s, a);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

// x (with W^T), w or d may be absent (C, dW, dg NULL).
static void f32_backward_blocks(const S2SArgs &x, const DWArgs &w, const RowDots &d, long long &w_blocks, long long &x_blocks, long long &d_blocks) {
  w_blocks = w.dW ? (long long)ceil_div(w.N, PT) * ceil_div(w.M, PT) * w.E : 0;
  x_blocks = x.C ? ((long long)ceil_div(x.Tk, PT) + x.E) * ceil_div(x.N, PT) : 0;
  d_blocks = d.dg ? ceil_div(d.Tk, 4) : 0;
}
// A dimension of a launch has less than 2^32 threads (the runtime takes more without an error and drops blocks).  The parts by
// themselves have two or three dimensions, or fewer blocks.
bool f32_backward_fits(const S2SArgs &x, const DWArgs &w, const RowDots &d) {
  long long w_blocks, x_blocks, d_blocks;
  f32_backward_blocks(x, w, d, w_blocks, x_blocks, d_blocks);
  return (w_blocks + x_blocks + d_blocks) * 256 < 1LL << 32;
}
int launch_f32_backward(hipStream_t s, const S2SArgs &x, const DWArgs &w, const RowDots &d) {
  long long w_blocks, x_blocks, d_blocks;
  f32_backward_blocks(x, w, d, w_blocks, x_blocks, d_blocks);
  if (!(w_blocks + x_blocks + d_blocks)) return SMOE_OK;
  const dim3 grid((unsigned)(w_blocks + x_blocks + d_blocks));
  const bool x_first = x_blocks && w_blocks && (long long)x.K * w.E > w.Tk;
  if (x.Hpre_in) hipLaunchKernelGGL(f32_backward_kernel<EPI_ACT_BWD>, grid, dim3(256), 0, s, x, w, d, (int)w_blocks, (int)x_blocks, x_first);
  else hipLaunchKernelGGL(f32_backward_kernel<EPI_NONE>, grid, dim3(256), 0, s, x, w, d, (int)w_blocks, (int)x_blocks, x_first);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
