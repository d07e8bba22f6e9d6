// Routing kernels: top-k gate (Sec. 3.1 step 1) and the stable bucket sort of the routed
// slots by expert (Sec. 3.1 step 2), integer-exact.
#include "common.h"
#include <limits.h>

// ---------------------------------------------------------------------------------------
// top-k gate: one thread per token.  Slot j takes the largest logit that comes after slot
// j-1's pick in the order (value descending, expert id ascending), so ties go to the lower
// id and no per-thread array is needed.  Gates are the softmax over the k picks.  A NaN logit
// counts as -inf (it can only be kept after every number), and picks that are all -inf share
// the weight equally, so every token writes all k slots whatever its logits hold.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) topk_gate_kernel(const float *__restrict__ logits, int T, int E, int k,
                                                        int32_t *__restrict__ idx, float *__restrict__ gates) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float *row = logits + (size_t)t * E;
  float prev_v = 0.f, first_v = 0.f, sum = 0.f;
  int prev_i = -1;
  for (int j = 0; j < k; ++j) {
    float best_v = 0.f;
    int best_i = -1;
    for (int e = 0; e < E; ++e) {
      float v = row[e];
      if (v != v) v = -INFINITY;
      bool after_prev = (prev_i < 0) || (v < prev_v) || (v == prev_v && e > prev_i);
      bool better = (best_i < 0) || (v > best_v);  // first hit wins ties -> lower id
      if (after_prev && better) { best_v = v; best_i = e; }
    }
    if (j == 0) first_v = best_v;
    float w = first_v == -INFINITY ? 1.0f : expf(best_v - first_v);
    idx[(size_t)t * k + j] = best_i;
    gates[(size_t)t * k + j] = w;
    sum += w;
    prev_v = best_v;
    prev_i = best_i;
  }
  float inv = 1.0f / sum;
  for (int j = 0; j < k; ++j) gates[(size_t)t * k + j] *= inv;
}

// Same selection with one wavefront per token for E <= 64 * VPL, by ranking: lane x holds logits x,
// x + 64, ...; the token's row sits in LDS and every lane counts, for each of its logits, how many
// come before it in the order (value descending, expert id ascending).  A logit of rank r < k is slot r.
template <int VPL>
__global__ void __launch_bounds__(256) topk_gate_wave_kernel(const float *__restrict__ logits, int T, int E, int k,
                                                             int32_t *__restrict__ idx, float *__restrict__ gates) {
  __shared__ __attribute__((aligned(16))) float rows[4][64 * VPL];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x * 4 + wave;
  if (t >= T) return;
  float *row = rows[wave];
  float v[VPL];
  int rank[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    int e = lane + 64 * i;
    // padding ranks after every real logit and never before one (-inf loses ties to the lower real ids)
    v[i] = e < E ? logits[(size_t)t * E + e] : -INFINITY;
    if (v[i] != v[i]) v[i] = -INFINITY;   // NaN counts as -inf
    row[e] = v[i];
    rank[i] = 0;
  }
  const int E4 = (E + 3) & ~3;   // the row is read four logits at a time; entries up to 64 * VPL are initialised
  for (int e0 = 0; e0 < E4; e0 += 4) {
    const float4 o4 = *reinterpret_cast<const float4 *>(row + e0);   // same address in every lane: a broadcast read
    const float o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < VPL; ++i) rank[i] += (o[c] > v[i]) || (o[c] == v[i] && e0 + c < lane + 64 * i);
  }
  // the rank-0 logit is the maximum; the gates are the softmax over the k kept logits
  float top = v[0];
#pragma unroll
  for (int i = 1; i < VPL; ++i) top = fmaxf(top, v[i]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) top = fmaxf(top, __shfl_xor(top, d, 64));
  float w[VPL], sum = 0.f;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    w[i] = (rank[i] < k && lane + 64 * i < E) ? (top == -INFINITY ? 1.0f : expf(v[i] - top)) : 0.f;
    sum += w[i];
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  const float inv = 1.0f / sum;
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (rank[i] < k && lane + 64 * i < E) {
      idx[(size_t)t * k + rank[i]] = lane + 64 * i;
      gates[(size_t)t * k + rank[i]] = w[i] * inv;
    }
}

// The same selection for few picks: k rounds of a wavefront maximum over order-preserving integer keys.  The ranking above
// compares every pair of a token's logits (64 experts: about 300 vector instructions, whatever k is); a round here is six
// cross-lane maxima (DPP, no LDS) and a ballot, about 14 instructions.
__device__ __forceinline__ int wave_max_i32(int v) {
  // rows of 16 lanes, then row 0 -> 1, 2 -> 3 (row_bcast:15) and the low half -> the high half (row_bcast:31); lane 63 holds the result
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x111, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x112, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x114, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x118, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x142, 0xa, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(v, 63);
}
template <int VPL>
__global__ void __launch_bounds__(256) topk_gate_rounds_kernel(const float *__restrict__ logits, int T, int E, int k,
                                                               int32_t *__restrict__ idx, float *__restrict__ gates) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  int key[VPL];   // signed order of the logits; INT_MIN lies below every logit's key: padding and picks already made
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int e = lane + 64 * i;
    float v = e < E ? logits[(size_t)t * E + e] : -INFINITY;
    v = v != v ? -INFINITY : v + 0.0f;            // NaN counts as -inf, -0 ties with +0
    const int b = __float_as_int(v);
    key[i] = e < E ? b ^ ((b >> 31) & 0x7fffffff) : INT_MIN;
  }
  int my_e = 0, my_key = INT_MIN;                 // lane j: the j-th pick
  for (int j = 0; j < k; ++j) {
    int best = key[0];
#pragma unroll
    for (int i = 1; i < VPL; ++i) best = max(best, key[i]);
    const int top = wave_max_i32(best);
    int e = -1;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {               // ascending ids: ties go to the lower one
      const unsigned long long at = __ballot(key[i] == top);
      if (e < 0 && at) e = 64 * i + __ffsll((long long)at) - 1;
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (lane + 64 * i == e) key[i] = INT_MIN;
    if (lane == j) { my_e = e; my_key = top; }
  }
  const float v = __int_as_float(my_key ^ ((my_key >> 31) & 0x7fffffff));
  const float top = __shfl(v, 0, 64);
  float w = lane < k ? (top == -INFINITY ? 1.0f : expf(v - top)) : 0.f;
  float sum = w;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  if (lane < k) {
    idx[(size_t)t * k + lane] = my_e;
    gates[(size_t)t * k + lane] = w / sum;
  }
}
// us at 32768 tokens, rounds / ranking: 64 experts k = 2 7.5 / 29.8, k = 8 12.2 / 29.9, k = 16 18.3 / 30.1 (the lines meet
// near k = 30); 256 experts k = 8 19.5 / 283.  A lane keeps one pick, so k <= 64.
static bool topk_by_rounds(int E, int k) { return k <= (E <= 64 ? 24 : 64); }

int launch_topk_gate(hipStream_t s, const float *logits, int T, int E, int k, int32_t *idx, float *gates) {
  if (T == 0) return SMOE_OK;
  dim3 grid(ceil_div(T, 4)), block(256);
  const bool rounds = topk_by_rounds(E, k);
  if (rounds && E <= 64)
    hipLaunchKernelGGL(topk_gate_rounds_kernel<1>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (rounds && E <= 128)
    hipLaunchKernelGGL(topk_gate_rounds_kernel<2>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (rounds && E <= 256)
    hipLaunchKernelGGL(topk_gate_rounds_kernel<4>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (rounds && E <= 1024)
    hipLaunchKernelGGL(topk_gate_rounds_kernel<16>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (E <= 64)
    hipLaunchKernelGGL(topk_gate_wave_kernel<1>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (E <= 128)
    hipLaunchKernelGGL(topk_gate_wave_kernel<2>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else if (E <= 256)
    hipLaunchKernelGGL(topk_gate_wave_kernel<4>, grid, block, 0, s, logits, T, E, k, idx, gates);
  else
    hipLaunchKernelGGL(topk_gate_kernel, dim3(ceil_div(T, 256)), dim3(256), 0, s, logits, T, E, k, idx, gates);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

// Gradient of the gate with respect to the router logits: softmax Jacobian on the k kept
// experts (g_j (dp_j - sum_i g_i dp_i)), zero elsewhere.  One thread per (token, expert)
// element so the [T,E] row is written whole and coalesced.
__global__ void __launch_bounds__(256) topk_gate_bwd_kernel(const int32_t *__restrict__ idx,
                                                            const float *__restrict__ gates,
                                                            const float *__restrict__ dgates, size_t total, int E, int k,
                                                            float *__restrict__ dlogits) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  size_t t = i / E;
  int e = (int)(i - t * E);
  const size_t base = t * k;
  float dot = 0.f, g_mine = 0.f, dp_mine = 0.f;
  for (int j = 0; j < k; ++j) {
    float g = gates[base + j], dp = dgates[base + j];
    dot += g * dp;
    if (idx[base + j] == e) { g_mine = g; dp_mine = dp; }
  }
  dlogits[i] = g_mine * (dp_mine - dot);
}

int launch_topk_gate_bwd(hipStream_t s, const int32_t *idx, const float *gates, const float *dgates, int T, int E, int k,
                         float *dlogits) {
  size_t total = (size_t)T * E;
  if (total == 0) return SMOE_OK;
  hipLaunchKernelGGL(topk_gate_bwd_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, idx, gates, dgates, total,
                     E, k, dlogits);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}

// ---------------------------------------------------------------------------------------
// Stable bucket sort by expert.  Slots are taken in chunks of 1024, one block each, a wavefront per 64 slots; a slot's place
// is (rows of earlier experts) + (rows of its expert in earlier chunks) + (in earlier wavefronts of its chunk) + (in lower
// lanes), the last one from ballots over the bits of the expert id.  Slots keep their order inside an expert because
// chunks, wavefronts and lanes are all counted in ascending slot order.  Everything here is latency: the data are a few
// hundred KB at most and a launch costs 3 to 5 us of the stream whatever it does, so the counts of the earlier chunks come
// from where fewest launches are needed (us for both kinds, top-k excluded; before: three launches of one-wavefront blocks):
//   one launch     (Tk <= ROUTE_ONE_LAUNCH) every block counts all slots itself, those before its chunk apart:
//                  6216 slots 21.2 -> 6.7, 16382 slots 15.1 -> 6.7, 32768 slots with 64 experts 21.8 -> 9.8;
//   two launches   (at most ROUTE_TWO_LAUNCH counters) a first kernel leaves one count per (expert, chunk), every block of
//                  the second adds up what it needs: 65536 slots 21.7 -> 10.5, 262144 slots 31.0 -> 15.6;
//   three launches (many experts times many chunks) a scan of the counters in between, so that it is done once.
// ---------------------------------------------------------------------------------------
static constexpr int ROUTE_CHUNK = 1024;            // slots (and threads) per block
static constexpr int ROUTE_WAVES = ROUTE_CHUNK / 64;
static constexpr int ROUTE_ONE_LAUNCH = 32768;
static constexpr int ROUTE_TWO_LAUNCH = 32768;
static constexpr int ROUTE_COPIES = 16;             // LDS histograms are kept in 16 copies, picked by lane, for up to
static constexpr int ROUTE_COPIES_MAX_E = 256;      // this many experts: popular experts otherwise serialise a wavefront's atomics

__device__ __forceinline__ int clamp_expert(int e, int E) { return e < 0 ? 0 : (e >= E ? E - 1 : e); }
__host__ __device__ inline int route_copies(int E, int threads) { return threads == ROUTE_CHUNK && E <= ROUTE_COPIES_MAX_E ? ROUTE_COPIES : 1; }

// rows of expert e in one of the LDS histograms
__device__ __forceinline__ int route_count_of(const int32_t *hist, int e, int copies) {
  int n = 0;
  for (int c = 0; c < copies; ++c) n += hist[e * copies + c];
  return n;
}

// total(e), before(e): rows of expert e over all slots and in the chunks before this block's (called by one thread per
// expert).  Leaves in next[e] the place of this chunk's first slot of expert e; block 0 writes the expert offsets.
template <int THREADS, typename TotalFn, typename BeforeFn>
__device__ __forceinline__ void route_first_places(int32_t *next, int E, int32_t *__restrict__ offsets, TotalFn total, BeforeFn before) {
  __shared__ int32_t s_wave[(THREADS / 64)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int run = 0;
  for (int e0 = 0; e0 < E; e0 += THREADS) {
    const int e = e0 + (int)threadIdx.x;
    const int n = e < E ? total(e) : 0, b = e < E ? before(e) : 0;
    int incl = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();          // also: every total and count has been read before `next` overwrites it
    int base = run;
    for (int w = 0; w < (THREADS / 64); ++w) {
      const int v = s_wave[w];
      if (w < wave) base += v;
      run += v;
    }
    if (e < E) {
      next[e] = base + incl - n + b;
      if (blockIdx.x == 0) offsets[e] = base + incl - n;
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) offsets[E] = run;
}

// Places this block's chunk; `e` is the (clamped) expert of the thread's slot.
template <int THREADS>
__device__ __forceinline__ void route_place_chunk(int32_t *next, int s, bool live, int e, int E, int32_t *__restrict__ sorted_e,
                                                  int32_t *__restrict__ sorted_s) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nbits = 32 - __clz(max(E - 1, 1));
  unsigned long long peers = __ballot(live);
  for (int b = 0; b < nbits; ++b) {
    const unsigned long long set = __ballot(live && ((e >> b) & 1));
    peers &= ((e >> b) & 1) ? set : ~set;
  }
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int rank = __popcll(peers & below), count = __popcll(peers);
  int pos = 0;
  for (int w = 0; w < THREADS / 64; ++w) {           // the wavefronts take their places in slot order
    if (w == wave && live) {
      pos = next[e] + rank;
      if (rank == 0) next[e] = pos + count;         // LDS operations of a wavefront execute in order: all its reads come first
    }
    __syncthreads();
  }
  if (live) {
    sorted_e[pos] = e;
    sorted_s[pos] = s;
  }
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS) route_one_launch_kernel(const int32_t *__restrict__ expert_idxs, int Tk, int E,
                                                                       int32_t *__restrict__ offsets, int32_t *__restrict__ sorted_e,
                                                                       int32_t *__restrict__ sorted_s) {
  extern __shared__ int32_t hist[];   // [2][E][copies]: slots before this block's chunk, the others
  const int copies = route_copies(E, THREADS), per = E * copies, copy = threadIdx.x & (copies - 1);
  const int base = blockIdx.x * THREADS, s = base + (int)threadIdx.x;
  const bool live = s < Tk;
  const int e = live ? clamp_expert(expert_idxs[s], E) : 0;
  for (int i = threadIdx.x; i < 2 * per; i += THREADS) hist[i] = 0;
  __syncthreads();
  constexpr int AHEAD = THREADS == ROUTE_CHUNK ? 8 : 1;   // loads in flight per thread
  for (int s0 = 0; s0 < Tk; s0 += AHEAD * THREADS) {
    int v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int q = s0 + u * THREADS + (int)threadIdx.x;
      v[u] = q < Tk ? expert_idxs[q] : -1;
    }
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int q = s0 + u * THREADS + (int)threadIdx.x;
      if (q < Tk) atomicAdd(&hist[(q < base ? 0 : per) + clamp_expert(v[u], E) * copies + copy], 1);
    }
  }
  __syncthreads();
  // `next` takes the place of the first histogram: [e] is written after all of row e and of the rows below it was read
  route_first_places<THREADS>(hist, E, offsets, [&](int x) { return route_count_of(hist, x, copies) + route_count_of(hist + per, x, copies); },
                     [&](int x) { return route_count_of(hist, x, copies); });
  route_place_chunk<THREADS>(hist, s, live, e, E, sorted_e, sorted_s);
}

__global__ void __launch_bounds__(ROUTE_CHUNK) route_count_kernel(const int32_t *__restrict__ expert_idxs, int Tk, int E,
                                                                  int32_t *__restrict__ counts /*[E][nchunk]*/) {
  extern __shared__ int32_t hist[];
  const int copies = route_copies(E, ROUTE_CHUNK);
  const int s = blockIdx.x * ROUTE_CHUNK + (int)threadIdx.x;
  const int e = s < Tk ? clamp_expert(expert_idxs[s], E) : 0;
  for (int i = threadIdx.x; i < E * copies; i += ROUTE_CHUNK) hist[i] = 0;
  __syncthreads();
  if (s < Tk) atomicAdd(&hist[e * copies + (threadIdx.x & (copies - 1))], 1);
  __syncthreads();
  // expert-major, so that what follows reads each expert's chunk counts contiguously
  for (int x = threadIdx.x; x < E; x += ROUTE_CHUNK) counts[(size_t)x * gridDim.x + blockIdx.x] = route_count_of(hist, x, copies);
}

// Second of two launches: the counts of all chunks are added up here, a wavefront per expert.
__global__ void __launch_bounds__(ROUTE_CHUNK) route_place_kernel(const int32_t *__restrict__ expert_idxs, int Tk, int E,
                                                                  const int32_t *__restrict__ counts /*[E][nchunk]*/,
                                                                  int32_t *__restrict__ offsets, int32_t *__restrict__ sorted_e,
                                                                  int32_t *__restrict__ sorted_s) {
  extern __shared__ int32_t sums[];   // [2][E]: rows in earlier chunks (then next place), in all chunks
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nchunk = gridDim.x;
  const int s = blockIdx.x * ROUTE_CHUNK + (int)threadIdx.x;
  const bool live = s < Tk;
  const int e = live ? clamp_expert(expert_idxs[s], E) : 0;
  for (int x = wave; x < E; x += ROUTE_WAVES) {
    int all = 0, before = 0;
    for (int c = lane; c < nchunk; c += 64) {
      const int n = counts[(size_t)x * nchunk + c];
      all += n;
      before += c < (int)blockIdx.x ? n : 0;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      all += __shfl_xor(all, d, 64);
      before += __shfl_xor(before, d, 64);
    }
    if (lane == 0) { sums[x] = before; sums[E + x] = all; }
  }
  __syncthreads();
  route_first_places<ROUTE_CHUNK>(sums, E, offsets, [&](int x) { return sums[E + x]; }, [&](int x) { return sums[x]; });
  route_place_chunk<ROUTE_CHUNK>(sums, s, live, e, E, sorted_e, sorted_s);
}

// Three launches: counts[e][c] -> start position of (chunk c, expert e); offsets[e] = rows before expert e.  One wavefront
// per expert at a time: lanes take chunks, a wave prefix sum orders them.
__global__ void __launch_bounds__(1024) route_scan_kernel(int32_t *__restrict__ counts, int nchunk, int E,
                                                          int32_t *__restrict__ offsets) {
  extern __shared__ int32_t totals[];  // [E] rows per expert, then exclusive prefix
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  for (int e = wave; e < E; e += nwave) {
    int sum = 0;
    for (int c = lane; c < nchunk; c += 64) sum += counts[(size_t)e * nchunk + c];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) totals[e] = sum;
  }
  __syncthreads();
  route_first_places<ROUTE_CHUNK>(totals, E, offsets, [&](int x) { return totals[x]; }, [](int) { return 0; });
  for (int e = wave; e < E; e += nwave) {
    int run = totals[e];
    for (int c0 = 0; c0 < nchunk; c0 += 64) {
      int c = c0 + lane;
      int n = (c < nchunk) ? counts[(size_t)e * nchunk + c] : 0;
      int incl = n;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
      }
      if (c < nchunk) counts[(size_t)e * nchunk + c] = run + incl - n;
      run += __shfl(incl, 63, 64);
    }
  }
}
__global__ void __launch_bounds__(ROUTE_CHUNK) route_place_scanned_kernel(const int32_t *__restrict__ expert_idxs, int Tk, int E,
                                                                          const int32_t *__restrict__ starts /*[E][nchunk]*/,
                                                                          int32_t *__restrict__ sorted_e, int32_t *__restrict__ sorted_s) {
  extern __shared__ int32_t next[];
  const int s = blockIdx.x * ROUTE_CHUNK + (int)threadIdx.x;
  const bool live = s < Tk;
  const int e = live ? clamp_expert(expert_idxs[s], E) : 0;
  for (int x = threadIdx.x; x < E; x += ROUTE_CHUNK) next[x] = starts[(size_t)x * gridDim.x + blockIdx.x];
  __syncthreads();
  route_place_chunk<ROUTE_CHUNK>(next, s, live, e, E, sorted_e, sorted_s);
}

// Scratch of the no-allocation routing entry point: the per-chunk expert counts that smoe_route keeps in
// caller workspace live here instead.  One copy per device, held until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress: kernels get the address looked up below.
static __device__ __align__(256) int32_t scratch[ROUTE_SCRATCH_BYTES / sizeof(int32_t)];

// Address of the current device's copy of the scratch array (called once per context, with the context's
// device current).
int route_scratch_address(int32_t **ptr) {
  void *p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SMOE_ERR_HIP;
  *ptr = (int32_t *)p;
  return SMOE_OK;
}

// Raises the dynamic LDS limit of the kernels that pass 64 KB together with their static arrays (once per context): two counters
// per expert, or one.
int init_route_kernels() {
  int rc = SMOE_OK;
  auto raise = [&](const void *kernel, size_t bytes) {
    if (rc == SMOE_OK && hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) rc = SMOE_ERR_HIP;
  };
  raise((const void *)route_one_launch_kernel<64>, 65536);
  raise((const void *)route_one_launch_kernel<256>, 65536);
  raise((const void *)route_one_launch_kernel<ROUTE_CHUNK>, (size_t)2 * ROUTE_MAX_E * sizeof(int32_t));
  raise((const void *)route_place_kernel, 65536);
  raise((const void *)route_scan_kernel, (size_t)ROUTE_MAX_E * sizeof(int32_t));
  return rc;
}

size_t route_workspace_bytes(int Tk, int E) {
  size_t nchunk = (size_t)ceil_div(Tk > 0 ? Tk : 1, ROUTE_CHUNK);
  return align256(nchunk * (size_t)E * sizeof(int32_t));
}

int launch_route(hipStream_t s, const int32_t *expert_idxs, int Tk, int E, int32_t *sorted_e, int32_t *sorted_s,
                 int32_t *offsets, void *ws) {
  const int nchunk = ceil_div(Tk > 0 ? Tk : 1, ROUTE_CHUNK);
  int32_t *counts = (int32_t *)ws;
  const size_t one = (size_t)E * sizeof(int32_t), hist = one * route_copies(E, ROUTE_CHUNK);
  // one chunk is always one launch, which leaves the scratch alone (up to 128 KB of LDS for two histograms)
  if (nchunk == 1 || (Tk <= ROUTE_ONE_LAUNCH && 2 * hist <= 65536)) {
    // a decoding batch fits one or four wavefronts, which start and meet sooner than sixteen (32 slots: 4.8 us with sixteen, 3.9 with
    // four); beyond 8192 experts their walk over the experts takes longer than the slots do
    if (Tk <= 64 && E <= 8192)
      hipLaunchKernelGGL(route_one_launch_kernel<64>, dim3(1), dim3(64), 2 * one, s, expert_idxs, Tk, E, offsets, sorted_e, sorted_s);
    else if (Tk <= 256 && E <= 8192)
      hipLaunchKernelGGL(route_one_launch_kernel<256>, dim3(1), dim3(256), 2 * one, s, expert_idxs, Tk, E, offsets, sorted_e, sorted_s);
    else
      hipLaunchKernelGGL(route_one_launch_kernel<ROUTE_CHUNK>, dim3(nchunk), dim3(ROUTE_CHUNK), 2 * hist, s, expert_idxs, Tk, E, offsets, sorted_e,
                         sorted_s);
    SMOE_LAUNCH_CHECK();
    return SMOE_OK;
  }
  hipLaunchKernelGGL(route_count_kernel, dim3(nchunk), dim3(ROUTE_CHUNK), hist, s, expert_idxs, Tk, E, counts);
  SMOE_LAUNCH_CHECK();
  if ((long long)E * nchunk <= ROUTE_TWO_LAUNCH && 2 * one <= 65536) {
    hipLaunchKernelGGL(route_place_kernel, dim3(nchunk), dim3(ROUTE_CHUNK), 2 * one, s, expert_idxs, Tk, E, counts, offsets, sorted_e, sorted_s);
    SMOE_LAUNCH_CHECK();
    return SMOE_OK;
  }
  hipLaunchKernelGGL(route_scan_kernel, dim3(1), dim3(1024), one, s, counts, nchunk, E, offsets);
  SMOE_LAUNCH_CHECK();
  if (Tk > 0) {
    hipLaunchKernelGGL(route_place_scanned_kernel, dim3(nchunk), dim3(ROUTE_CHUNK), one, s, expert_idxs, Tk, E, counts, sorted_e, sorted_s);
    SMOE_LAUNCH_CHECK();
  }
  return SMOE_OK;
}
