// Memory-bound row kernels around the grouped GEMMs: the activation of Alg. 3, the weighted
// sum over a token's k slots (Alg. 1), the `group` copy and the routing-weight gradient of
// Alg. 2.  All read/write 16 bytes per lane when the row width allows it.
#include "common.h"
#include <type_traits>

template <typename T> struct Vec16 { static constexpr int N = 16 / sizeof(T); T v[N]; } __attribute__((aligned(16)));

template <typename T> __device__ __forceinline__ void load_vec(const T *p, float (&f)[16 / sizeof(T)]) {
  Vec16<T> r = *reinterpret_cast<const Vec16<T> *>(p);
#pragma unroll
  for (int i = 0; i < Vec16<T>::N; ++i) f[i] = to_f32<T>(r.v[i]);
}
template <typename T> __device__ __forceinline__ void store_vec(T *p, const float (&f)[16 / sizeof(T)]) {
  Vec16<T> r;
#pragma unroll
  for (int i = 0; i < Vec16<T>::N; ++i) r.v[i] = from_f32<T>(f[i]);
  *reinterpret_cast<Vec16<T> *>(p) = r;
}

typedef uint32_t raw16 __attribute__((ext_vector_type(4)));
// read once and dead afterwards: no line is kept (combine of 262144 rows of 8 KB: 459 -> 403 us, 6.0 TB/s)
template <typename T> __device__ __forceinline__ Vec16<T> load_once(const T *p) {
  const raw16 r = __builtin_nontemporal_load(reinterpret_cast<const raw16 *>(p));
  return __builtin_bit_cast(Vec16<T>, r);
}

// How a block's threads are laid over rows of `per_row` 16-byte chunks, chosen on the host so that no thread divides: rows
// of up to 64 chunks get the next power of two lanes each, longer ones one to four whole wavefronts that walk the row
// together.  (With one chunk per thread numbered through the tensor, the 64-bit division of that number cost more than the
// 16 bytes it located: 65536 sorted rows of 4 KB were grouped at 3.8 TB/s.)
struct RowLanes {
  int shift;     // thread >> shift = row inside the block
  int lanes;     // threads of a row
  int rows;      // rows side by side in a block
};
static RowLanes row_lanes(int per_row) {
  RowLanes l{0, 1, 256};
  while (l.lanes < per_row && l.lanes < 64) {
    ++l.shift;
    l.lanes *= 2;
    l.rows /= 2;
  }
  if (per_row > 64) {
    const int waves = per_row > 192 ? 4 : (per_row + 63) / 64;
    l.lanes = 64 * waves;
    l.rows = waves == 2 ? 2 : 1;
    l.shift = waves == 2 ? 7 : 8;
  }
  return l;
}

static int row_blocks(long long rows, int per_block) {
  const long long b = (rows + per_block - 1) / per_block;
  return (int)(b < 256 * 64 ? b : 256 * 64);
}

// ---- activation forward: H = act(Hpre)
template <typename T, int ACT>
__global__ void __launch_bounds__(256) act_fwd_kernel(const T *__restrict__ Hpre, T *__restrict__ H, int rows,
                                                      int d_expert, RowLanes l) {
  constexpr int V = 16 / sizeof(T);
  const int d_h = (ACT == SMOE_ACT_SWIGLU) ? 2 * d_expert : d_expert;
  const int lane = (int)threadIdx.x & (l.shift == 8 ? 255 : l.lanes - 1);
  for (long long r = (long long)blockIdx.x * l.rows + ((int)threadIdx.x >> l.shift); r < rows; r += (long long)gridDim.x * l.rows)
  for (int c = lane * V; c < d_expert; c += l.lanes * V) {
    float a[V], out[V];
    load_vec<T>(Hpre + r * d_h + c, a);
    if (ACT == SMOE_ACT_SWIGLU) {
      float u[V];
      load_vec<T>(Hpre + r * d_h + d_expert + c, u);
#pragma unroll
      for (int i = 0; i < V; ++i) out[i] = a[i] * sigmoid_f(a[i]) * u[i];
    } else if (ACT == SMOE_ACT_GELU) {
#pragma unroll
      for (int i = 0; i < V; ++i) out[i] = gelu_f(a[i]);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) out[i] = a[i];
    }
    store_vec<T>(H + r * d_expert + c, out);
  }
}

// ---- activation backward: dHpre = act'(Hpre) * dH.
template <typename T, int ACT>
__global__ void __launch_bounds__(256) act_bwd_kernel(const T *__restrict__ Hpre, const T *__restrict__ dH,
                                                      T *__restrict__ dHpre, int rows, int d_expert, RowLanes l) {
  constexpr int V = 16 / sizeof(T);
  const int d_h = (ACT == SMOE_ACT_SWIGLU) ? 2 * d_expert : d_expert;
  const int lane = (int)threadIdx.x & (l.shift == 8 ? 255 : l.lanes - 1);
  for (long long r = (long long)blockIdx.x * l.rows + ((int)threadIdx.x >> l.shift); r < rows; r += (long long)gridDim.x * l.rows)
  for (int c = lane * V; c < d_expert; c += l.lanes * V) {
    float a[V], g[V], o1[V];
    load_vec<T>(Hpre + r * d_h + c, a);
    load_vec<T>(dH + r * d_expert + c, g);
    if (ACT == SMOE_ACT_SWIGLU) {
      float u[V], o2[V];
      load_vec<T>(Hpre + r * d_h + d_expert + c, u);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        float sg = sigmoid_f(a[i]);
        float silu = a[i] * sg;
        o1[i] = g[i] * u[i] * (sg + silu * (1.0f - sg));
        o2[i] = g[i] * silu;
      }
      store_vec<T>(dHpre + r * d_h + c, o1);
      store_vec<T>(dHpre + r * d_h + d_expert + c, o2);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) o1[i] = (ACT == SMOE_ACT_GELU) ? g[i] * gelu_grad_f(a[i]) : g[i];
      store_vec<T>(dHpre + r * d_h + c, o1);
    }
  }
}

// ---- weighted sum over a token's k slots: Y[t] = sum_j g[t*k+j] * Yhat[t*k+j] + more[0][t] + more[1][t]  (g may be null = 1,
// and both arrays of `more`)
// Bound by HBM (the k slot rows are read once): K rows are in flight at once, all of them up to k = 8, and past the caches.  65536
// rows of 4 KB: k = 3 61.5 -> 54.5 us, 5 59.5 -> 52, 6 59.5 -> 50.5, 7 57 -> 50.5, 12 56 -> 49.5 (one row at a time, through the
// caches, before); k = 2, 4 and 8 61, 53 and 50.
template <typename T, int K>
__global__ void __launch_bounds__(256) combine_kernel(const T *__restrict__ Yhat, const float *__restrict__ g,
                                                      T *__restrict__ Y, int T_rows, int k, int d, RowLanes l,
                                                      const T *__restrict__ more0, const T *__restrict__ more1) {
  constexpr int V = 16 / sizeof(T);
  const int lane = (int)threadIdx.x & (l.shift == 8 ? 255 : l.lanes - 1);
  for (long long t = (long long)blockIdx.x * l.rows + ((int)threadIdx.x >> l.shift); t < T_rows; t += (long long)gridDim.x * l.rows) {
    const T *in = Yhat + t * k * d;
    const float *gt = g ? g + t * k : nullptr;
    for (int c = lane * V; c < d; c += l.lanes * V) {
      float acc[V];
#pragma unroll
      for (int i = 0; i < V; ++i) acc[i] = 0.f;
      auto add = [&](int j, const Vec16<T> &row) {
        const float gj = gt ? gt[j] : 1.0f;
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = fmaf(gj, to_f32<T>(row.v[i]), acc[i]);
      };
      int j = 0;
      for (; j + K <= k; j += K) {
        Vec16<T> rows[K];
#pragma unroll
        for (int u = 0; u < K; ++u) rows[u] = load_once<T>(in + (size_t)(j + u) * d + c);
#pragma unroll
        for (int u = 0; u < K; ++u) add(j + u, rows[u]);
      }
      for (; j < k; ++j) add(j, load_once<T>(in + (size_t)j * d + c));
      if (more0) {
        float a[V], b[V];
        load_vec<T>(more0 + t * d + c, a);
        load_vec<T>(more1 + t * d + c, b);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] += a[i] + b[i];
      }
      store_vec<T>(Y + t * d + c, acc);
    }
  }
}

// ---- group: out[i] = g[o[i]] * in[o[i] / fan]  (g may be null = 1).  GROUP_ROWS rows per thread at a time: their loads are in
// flight together.
constexpr int GROUP_ROWS = 4;
template <typename T>
__global__ void __launch_bounds__(256) group_kernel(const T *__restrict__ in, const int32_t *__restrict__ o, int fan,
                                                    const float *__restrict__ g, T *__restrict__ out, int Tk, int d, RowLanes l) {
  constexpr int V = 16 / sizeof(T);
  const int lane = (int)threadIdx.x & (l.shift == 8 ? 255 : l.lanes - 1), sub = (int)threadIdx.x >> l.shift;
  const long long step = (long long)gridDim.x * l.rows * GROUP_ROWS;
  for (long long i0 = (long long)blockIdx.x * l.rows * GROUP_ROWS + sub; i0 < Tk; i0 += step) {
    const T *src[GROUP_ROWS];
    float gs[GROUP_ROWS];
    int slot[GROUP_ROWS];
#pragma unroll
    for (int u = 0; u < GROUP_ROWS; ++u) slot[u] = o[min(i0 + u * l.rows, (long long)Tk - 1)];
#pragma unroll
    for (int u = 0; u < GROUP_ROWS; ++u) {
      src[u] = in + (size_t)((unsigned)slot[u] / (unsigned)fan) * d;
      gs[u] = g ? g[slot[u]] : 1.0f;
    }
    for (int c = lane * V; c < d; c += l.lanes * V) {
      Vec16<T> a[GROUP_ROWS];
#pragma unroll
      for (int u = 0; u < GROUP_ROWS; ++u) a[u] = *reinterpret_cast<const Vec16<T> *>(src[u] + c);
#pragma unroll
      for (int u = 0; u < GROUP_ROWS; ++u) {
        if (i0 + u * l.rows >= Tk) break;
        if (g)
#pragma unroll
          for (int q = 0; q < V; ++q) a[u].v[q] = from_f32<T>(to_f32<T>(a[u].v[q]) * gs[u]);
        *reinterpret_cast<Vec16<T> *>(out + (size_t)(i0 + u * l.rows) * d + c) = a[u];
      }
    }
  }
}

// ---- inv[o[i]] = i, the sorted position of every slot
__global__ void __launch_bounds__(256) invert_kernel(const int32_t *__restrict__ o, int32_t *__restrict__ inv, int Tk) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < Tk) inv[o[i]] = i;
}

// ---- spread: the copy `group` makes, from the side of the source: out[inv[t * fan + j]] = g[t * fan + j] * in[t].  Bound by the
// write of the Tk rows; `group` read every source row fan times as well, from whichever XCD's L2 its sorted row fell to.
struct Spread {
  const bf16_t *in;
  const float *g;
  bf16_t *out;
  int rows, d, blocks;   // blocks 0: nothing to do
  RowLanes l;
};
template <int K>   // fan where it is at most 8 (its stores then need no loop: k = 2 65 -> 63.5 us, k = 4 52.5 -> 51), else 0
__device__ __forceinline__ void spread_rows(const Spread &s, const int32_t *__restrict__ inv, int fan_any, int block) {
  const int fan = K ? K : fan_any;
  const int lane = (int)threadIdx.x & (s.l.shift == 8 ? 255 : s.l.lanes - 1);
  for (long long t = (long long)block * s.l.rows + ((int)threadIdx.x >> s.l.shift); t < s.rows; t += (long long)s.blocks * s.l.rows) {
    const int32_t *pos = inv + t * fan;
    const float *gt = s.g ? s.g + t * fan : nullptr;
    int32_t at[K ? K : 1];                     // read once: the compiler cannot know that the copies do not lie over them
    float weight[K ? K : 1];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      at[j] = pos[j];
      weight[j] = gt ? gt[j] : 1.0f;
    }
    for (int c = lane * 8; c < s.d; c += s.l.lanes * 8) {
      const Vec16<bf16_t> a = *reinterpret_cast<const Vec16<bf16_t> *>(s.in + t * s.d + c);
#pragma unroll
      for (int j = 0; j < (K ? K : fan); ++j) {
        Vec16<bf16_t> v = a;
        if (gt) {
          const float gs = K ? weight[j] : gt[j];
#pragma unroll
          for (int q = 0; q < 8; ++q) v.v[q] = (bf16_t)((float)a.v[q] * gs);
        }
        *reinterpret_cast<Vec16<bf16_t> *>(s.out + (size_t)(K ? at[j] : pos[j]) * s.d + c) = v;
      }
    }
  }
}
// Up to two such copies of the same fan and the row dots of dp in one launch: none waits for another, and a launch of its own is 4 us
// of start and end (16396 rows, 2048 -> 1536, k = 4: 12.4 + 13.0 + 14.8 us and two gaps -> 35.8 us; the training step 421.6 -> 413.0).
template <int K>
__global__ void __launch_bounds__(256) spread_kernel(Spread a, Spread b, RowDots dots, const int32_t *__restrict__ inv, int fan) {
  int block = blockIdx.x;
  if (block < a.blocks) return spread_rows<K>(a, inv, fan, block);
  block -= a.blocks;
  if (block < b.blocks) return spread_rows<K>(b, inv, fan, block);
  block -= b.blocks;
  const int s = block * 4 + ((int)threadIdx.x >> 6);
  if (s < dots.Tk) row_dot<bf16_t>(dots, s, threadIdx.x & 63);
}

// ---- dg[o[i]] = sum_c part[i, c] (and inv[o[i]] = i, inv may be null): eight lanes per sorted row, each adds the pairs of slabs lane, lane + 8, ... in ascending
// order, then a fixed tree (a thread per row read its 448 bytes at a stride: 23 us for 32768 rows of 112 slabs)
__global__ void __launch_bounds__(256) dp_reduce_kernel(const float2 *__restrict__ part, int ld2, const int32_t *__restrict__ o,
                                                        float *__restrict__ dg, int32_t *__restrict__ inv, int Tk) {
  const int i = blockIdx.x * 32 + ((int)threadIdx.x >> 3), lane = (int)threadIdx.x & 7;
  const float2 *p = part + (size_t)min(i, Tk - 1) * ld2;
  float acc = 0.f;
  for (int c = lane; c < ld2; c += 8) acc += p[c].x + p[c].y;
#pragma unroll
  for (int off = 4; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0 && i < Tk) {
    const int slot = o[i];
    dg[slot] = acc;
    if (inv) inv[slot] = i;
  }
}

// ---- dg[s] = <dY[s / kp], Yhat[s]> : one wavefront per slot, lanes stride the row.
template <typename T> __global__ void __launch_bounds__(256) rowdot_kernel(RowDots r) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s < r.Tk) row_dot<T>(r, s, threadIdx.x & 63);
}

// -----------------------------------------------------------------------------------------
static inline int grid_for(size_t work_items) {
  size_t b = (work_items + 255) / 256;
  if (b > 256 * 64) b = 256 * 64;
  return (int)(b ? b : 1);
}
template <typename T> static bool vec_ok(int d) { return d % (16 / (int)sizeof(T)) == 0; }

// bf16 only: the fp32 products apply the activation and its derivative in their epilogues
int launch_act_fwd(hipStream_t s, smoe_act act, const void *Hpre, void *H, int rows, int d_expert) {
  if (!vec_ok<bf16_t>(d_expert)) return SMOE_ERR_UNSUPPORTED;
  if (rows < 1) return SMOE_OK;
  const RowLanes l = row_lanes(d_expert / 8);
  const dim3 g(row_blocks(rows, l.rows)), b(l.lanes * l.rows);
  const bf16_t *in = (const bf16_t *)Hpre;
  bf16_t *out = (bf16_t *)H;
  if (act == SMOE_ACT_SWIGLU) hipLaunchKernelGGL((act_fwd_kernel<bf16_t, SMOE_ACT_SWIGLU>), g, b, 0, s, in, out, rows, d_expert, l);
  else if (act == SMOE_ACT_GELU) hipLaunchKernelGGL((act_fwd_kernel<bf16_t, SMOE_ACT_GELU>), g, b, 0, s, in, out, rows, d_expert, l);
  else hipLaunchKernelGGL((act_fwd_kernel<bf16_t, SMOE_ACT_NONE>), g, b, 0, s, in, out, rows, d_expert, l);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
int launch_act_bwd(hipStream_t s, smoe_act act, const void *Hpre, const void *dH, void *dHpre, int rows, int d_expert) {
  if (!vec_ok<bf16_t>(d_expert)) return SMOE_ERR_UNSUPPORTED;
  if (rows < 1) return SMOE_OK;
  const RowLanes l = row_lanes(d_expert / 8);
  const dim3 g(row_blocks(rows, l.rows)), b(l.lanes * l.rows);
  const bf16_t *a = (const bf16_t *)Hpre, *gr = (const bf16_t *)dH;
  bf16_t *out = (bf16_t *)dHpre;
  if (act == SMOE_ACT_SWIGLU) hipLaunchKernelGGL((act_bwd_kernel<bf16_t, SMOE_ACT_SWIGLU>), g, b, 0, s, a, gr, out, rows, d_expert, l);
  else if (act == SMOE_ACT_GELU) hipLaunchKernelGGL((act_bwd_kernel<bf16_t, SMOE_ACT_GELU>), g, b, 0, s, a, gr, out, rows, d_expert, l);
  else hipLaunchKernelGGL((act_bwd_kernel<bf16_t, SMOE_ACT_NONE>), g, b, 0, s, a, gr, out, rows, d_expert, l);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

// calls f with k as a constant, or 8 where it is larger
template <typename F> static void with_rows(int k, F f) {
  switch (k) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{});
  }
}

template <typename T>
static int combine_t(hipStream_t s, const void *Yhat, const float *g, void *Y, int T_rows, int k, int d, const void *m0, const void *m1) {
  if (!vec_ok<T>(d)) return SMOE_ERR_UNSUPPORTED;
  if (T_rows < 1) return SMOE_OK;
  const RowLanes l = row_lanes(d / (16 / (int)sizeof(T)));
  const int blocks = row_blocks(T_rows, l.rows);
  with_rows(k, [&](auto rows) {
    hipLaunchKernelGGL((combine_kernel<T, decltype(rows)::value>), dim3(blocks), dim3(l.lanes * l.rows), 0, s, (const T *)Yhat, g, (T *)Y, T_rows,
                       k, d, l, (const T *)m0, (const T *)m1);
  });
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
int launch_combine(hipStream_t s, smoe_dtype dt, const void *Yhat, const float *g, void *Y, int T, int k, int d, const void *more0,
                   const void *more1) {
  return dt == SMOE_BF16 ? combine_t<bf16_t>(s, Yhat, g, Y, T, k, d, more0, more1) : combine_t<float>(s, Yhat, g, Y, T, k, d, more0, more1);
}

template <typename T>
static int group_t(hipStream_t s, const void *in, const int32_t *o, int fan, const float *g, void *out, int Tk, int d) {
  if (!vec_ok<T>(d)) return SMOE_ERR_UNSUPPORTED;
  if (Tk < 1) return SMOE_OK;
  const RowLanes l = row_lanes(d / (16 / (int)sizeof(T)));
  hipLaunchKernelGGL((group_kernel<T>), dim3(row_blocks(Tk, l.rows * GROUP_ROWS)), dim3(l.lanes * l.rows), 0, s, (const T *)in, o, fan, g,
                     (T *)out, Tk, d, l);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
int launch_group(hipStream_t s, smoe_dtype dt, const void *in, const int32_t *o, int fan, const float *g, void *out, int Tk, int d) {
  return dt == SMOE_BF16 ? group_t<bf16_t>(s, in, o, fan, g, out, Tk, d) : group_t<float>(s, in, o, fan, g, out, Tk, d);
}

int launch_invert(hipStream_t s, const int32_t *o, int32_t *inv, int Tk) {
  if (Tk < 1) return SMOE_OK;
  hipLaunchKernelGGL(invert_kernel, dim3(ceil_div(Tk, 256)), dim3(256), 0, s, o, inv, Tk);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
static Spread spread_of(const void *in, const float *g, void *out, int rows, int d) {
  const RowLanes l = row_lanes(d / 8);
  return Spread{(const bf16_t *)in, g, (bf16_t *)out, rows, d, row_blocks(rows, l.rows), l};
}
int launch_spread(hipStream_t s, const void *in, const int32_t *inv, int fan, const float *g, void *out, int Tk, int d, const RowDots &dots, const void *in2,
                  void *out2, int d2) {
  if (!vec_ok<bf16_t>(d) || (in2 && !vec_ok<bf16_t>(d2)) || (dots.dg && !vec_ok<bf16_t>(dots.d))) return SMOE_ERR_UNSUPPORTED;
  if (Tk < 1) return SMOE_OK;
  const Spread a = spread_of(in, g, out, Tk / fan, d), b = in2 ? spread_of(in2, nullptr, out2, Tk / fan, d2) : Spread{};
  auto launch = [&](auto k) {
    hipLaunchKernelGGL(spread_kernel<decltype(k)::value>, dim3(a.blocks + b.blocks + (dots.dg ? ceil_div(dots.Tk, 4) : 0)), dim3(256), 0, s, a, b, dots, inv, fan);
  };
  if (fan <= 8) with_rows(fan, launch);
  else launch(std::integral_constant<int, 0>{});
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

int launch_dp_reduce(hipStream_t s, const float *part, int ld, const int32_t *o, float *dg, int32_t *inv, int Tk) {
  if (!Tk) return SMOE_OK;
  if (ld % 2) return SMOE_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(dp_reduce_kernel, dim3(ceil_div(Tk, 32)), dim3(256), 0, s, (const float2 *)part, ld / 2, o, dg, inv, Tk);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

template <typename T>
static int rowdot_t(hipStream_t s, const void *dY, const void *Yhat, float *dg, int Tk, int kp, int d) {
  if (!vec_ok<T>(d)) return SMOE_ERR_UNSUPPORTED;
  if (!Tk) return SMOE_OK;
  hipLaunchKernelGGL((rowdot_kernel<T>), dim3(ceil_div(Tk, 4)), dim3(256), 0, s, RowDots{dY, Yhat, dg, Tk, kp, d});
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
int launch_rowdot(hipStream_t s, smoe_dtype dt, const void *dY, const void *Yhat, float *dg, int Tk, int kp, int d) {
  return dt == SMOE_BF16 ? rowdot_t<bf16_t>(s, dY, Yhat, dg, Tk, kp, d) : rowdot_t<float>(s, dY, Yhat, dg, Tk, kp, d);
}

// ------------------------------------------------------------------------------------------
// helpers of the attention layer: offsets of one all-rows segment (a dense product runs through
// the grouped kernels as one expert), and the sum of three bf16 arrays
// ------------------------------------------------------------------------------------------
__global__ void dense_offsets_kernel(int32_t *off, int n) {
  if (threadIdx.x == 0) { off[0] = 0; off[1] = n; }
}
int launch_dense_offsets(hipStream_t s, int32_t *off, int n) {
  hipLaunchKernelGGL(dense_offsets_kernel, dim3(1), dim3(64), 0, s, off, n);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

__global__ void __launch_bounds__(256) add3_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ b,
                                                   const bf16_t *__restrict__ c, bf16_t *__restrict__ out, size_t n8) {
  typedef bf16_t v8 __attribute__((ext_vector_type(8)));
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
    v8 x = reinterpret_cast<const v8 *>(a)[i], y = reinterpret_cast<const v8 *>(b)[i], z = reinterpret_cast<const v8 *>(c)[i], r;
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q] = (bf16_t)((float)x[q] + (float)y[q] + (float)z[q]);
    reinterpret_cast<v8 *>(out)[i] = r;
  }
}
int launch_add3(hipStream_t s, const void *a, const void *b, const void *c, void *out, size_t n) {
  if (n % 8) return SMOE_ERR_UNSUPPORTED;
  if (!n) return SMOE_OK;
  hipLaunchKernelGGL(add3_kernel, dim3(grid_for(n / 8)), dim3(256), 0, s, (const bf16_t *)a, (const bf16_t *)b,
                     (const bf16_t *)c, (bf16_t *)out, n / 8);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
