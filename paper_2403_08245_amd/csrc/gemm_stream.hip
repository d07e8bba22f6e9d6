// Persistent ("stream") form of the bf16 matrix-core grouped GEMMs.
//
// Blocks walk lists of output tiles.  The LDS ring of the contraction loop never drains between tiles: the loader runs
// ahead of the multiplying side and simply moves on to the next tile's operand rows, so the next tile's first stages land
// while the current tile is being finished and written out.
//
// scatter2scatter: a stage is 64 contraction elements, so that an operand row whose elements are contiguous (rows of X and dY,
// and of W in the W^T products) is fetched as one whole 128-byte cache line.  In pieces of 64 bytes, half a line a stage, L2
// delivered every line twice (it was gone from the 32 KB L1 by then): with all compute units at it 67 bytes per ns and unit from
// L2 instead of 134, and 35.8 M line requests in a W^T product whose operands are 18.9 M lines.
// A stage has four phases of 16 elements.  The first two multiply fragments that are in registers already and read those of
// the stage's other three sixteenths behind them; after them every wavefront holds all of the stage's fragments, so its slot is
// free and the third and fourth phase, which only multiply, issue the loads that refill it.  The fourth also reads the
// next stage's first fragments.  So a ring of S slots has S - 1/2 stages of loads in flight at most and S - 3/4 at least.
// The loads are spread over two phases: all in one (64 KB a compute unit in 512 cycles) the wavefronts stand behind the memory
// pipeline with their matrix instructions (32768 rows, 14336 -> 4096: 3008 -> 3382 us).
//
// Two shapes (Shape below), one block per compute unit, one wavefront per SIMD:
//   Big   256 x 256 tiles, two slots of 64 KB, 256 accumulators: the fewest operand bytes per multiply-add.
//   Half  128 x 256 tiles, three slots of 48 KB, 128 accumulators: half as many rows per tile waste fewer rows at segment ends and
//         leave less work over when the tiles do not fill a last round; the price is 1.5 times the operand traffic.  HalfShort has two
//         slots, for the short launches that launch_s2s_cfg names.
// Measured, stages of 32 elements (there with two blocks per compute unit for the 128 x 256 tiles) / these, in us: W^T products of
// 32768 rows, 28672 -> 4096: 6420 / 5800; 65536 rows in 64 experts, 1024 -> 2048: 306 / 287; 8192 rows in 8 experts, 5632 -> 1024:
// 120 / 106; 6002 rows, 6832 -> 1280 (rows of W that start off the lines): 200 / 120.  W as stored, where only the rows of X gain:
// 4096 -> 2 x 14336 with SwiGLU 6370 / 6240, 14336 -> 4096: 3034 / 3025, 65536 rows, 2048 -> 2 x 512: 274 / 268.
//
// groupXTY runs the same stages on Big tiles.  Its operand rows are 512 contiguous bytes a tile, so the lines are not what it gains;
// half the barriers are: 16396 rows in 16 experts, 2048 x 1536: 97 -> 93 us, 8192 rows in 8 experts, 1024 x 5632: 94 -> 89, and long
// segments the same (32768 rows, 4096 x 28672: 6.04 ms).
//
// Loads are inline assembly so that the waits are placed by hand; stores share the hardware counter with them and complete
// in order, and because every epilogue issues a known number of stores at least, the first wait after an epilogue steps
// over them instead of sitting out their acknowledgement.  All loads go through range-checked buffer windows: rows past a
// segment and contraction elements past K read zeros.  Row indices travel through LDS by direct-to-LDS loads as well: no
// ordinary global load sits in the loop, so the compiler never inserts a full wait in front of the loads in flight.
#include "gemm_epilogue.h"
#include <type_traits>

namespace {

constexpr int SK = 64;                                  // contraction elements per stage: 128 bytes, one cache line
constexpr int B_BYTES = TB * SK * 2;                    // W (256 columns) part of a stage

template <int FM_, int SLOTS_, bool ONCE_ = false> struct Shape {
  static constexpr int FM = FM_;                        // 32-row fragments per wavefront (2 x 2 wavefronts, FR = 4 column fragments)
  static constexpr int TM = FM * 64;                    // tile rows; tile columns are TB = 256
  static constexpr int A_BYTES = TM * SK * 2;
  static constexpr int SLOTS = SLOTS_;
  static constexpr bool ONCE = ONCE_;                   // W is read past the caches
  static constexpr int NLA = A_BYTES / 4096;            // load instructions per wavefront and stage: A part,
  static constexpr int NLB = B_BYTES / 4096;            // W part,
  static constexpr int NL = NLA + NLB;                  // both
  static constexpr int NF = FM + FR;                    // fragments per wavefront and 16 contraction elements
  static constexpr int PART = TM * TB;                  // elements of an fp32 partial tile
  static constexpr int RING_BYTES = SLOTS * (A_BYTES + B_BYTES);   // A slots, then W slots
  // Where the ring leaves no LDS for it, the patch of an epilogue is the part of the finished slot that the wavefront loads
  // itself: nobody else touches it until the same wavefront issues that slot's next loads, held back until after the epilogue.
  static constexpr bool PATCH_IN_SLOT = RING_BYTES > 140 * 1024;
  static constexpr int LDS_BYTES = RING_BYTES + (PATCH_IN_SLOT ? 0 : 4 * EPI_WAVE_BYTES);
};
using Big = Shape<4, 2>;
using Half = Shape<2, 3>;
using HalfOnce = Shape<2, 3, true>;
using HalfShort = Shape<2, 2>;
using HalfShortOnce = Shape<2, 2, true>;
constexpr int MAX_STREAM_GRID = 256;                    // compute units used; the partial-tile scratch holds this many big tiles

template <typename S> struct Frags {                    // one wavefront's fragments for 16 contraction elements
  bf16x8 a[S::FM], b[FR];
};
// item I of a set of fragments, in the order the products consume them: b0 a0 b1 b2 b3 a1 (a2 a3)
template <typename S, typename Ops>
__device__ __forceinline__ void read_item(const Ops &ops, Frags<S> &f, int item, const char *a_slot, const char *b_slot, int kk) {
  if (item == 0) f.b[0] = ops.frag_b(b_slot, 0, kk);
  else if (item == 1) f.a[0] = ops.frag_a(a_slot, 0, kk);
  else if (item < FR + 1) f.b[item - 1] = ops.frag_b(b_slot, item - 1, kk);
  else f.a[item - FR] = ops.frag_a(a_slot, item - FR, kk);
}
// The products of 16 contraction elements; read(m) and load(m) issue the LDS reads and the loads that go behind fragment row m.
// FIRST: the tile's first products overwrite the accumulators.
template <bool FIRST, typename S, typename ReadFn, typename LoadFn>
__device__ __forceinline__ void phase(const Frags<S> &use, f32x16 (&acc)[S::FM][FR], ReadFn read, LoadFn load) {
  f32x16 zero;
#pragma unroll
  for (int q = 0; q < 16; ++q) zero[q] = 0.f;
  sched_fence();
#pragma unroll
  for (int m = 0; m < S::FM; ++m) {
#pragma unroll
    for (int n = 0; n < FR; ++n)
      acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(use.b[n], use.a[m], FIRST ? zero : acc[m][n], 0, 0, 0);
    read(m);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
    }
    sched_fence();
    load(m);
    sched_fence();
  }
}
// One stage of 64 contraction elements in slot `cur`, the next one in slot `nxt`.  f[kk]: fragments of 16 elements each; f[0] is in
// registers on entry, and the next stage's on exit.  STORES: that many stores were issued after the next stages' loads at least.
// LAST with the patch in the slot: the refill is left to the caller.
template <bool FIRST, bool LAST, int STORES, typename S, typename Ops, typename Slot, typename Next>
__device__ __forceinline__ void stage_step(const Ops &ops, Frags<S> (&f)[4], f32x16 (&acc)[S::FM][FR], const char *smem, uint32_t lds0, Slot cur,
                                           Next nxt) {
  constexpr int NF = S::NF, HEAD = NF / 2;
  constexpr bool FILL = !(LAST && S::PATCH_IN_SLOT);
  const char *a = smem + (uint32_t)cur * S::A_BYTES, *b = smem + S::SLOTS * S::A_BYTES + (uint32_t)cur * B_BYTES;
  const char *an = smem + (uint32_t)nxt * S::A_BYTES, *bn = smem + S::SLOTS * S::A_BYTES + (uint32_t)nxt * B_BYTES;
  const uint32_t fill_a = lds0 + (uint32_t)cur * S::A_BYTES, fill_b = lds0 + S::SLOTS * S::A_BYTES + (uint32_t)cur * B_BYTES;
  auto none = [](int) {};
  // reads of the first two phases: f[1], f[2] and f[3]
  auto early = [&](int from, int to) {
#pragma unroll
    for (int i = 0; i < 3 * NF; ++i)
      if (i >= from && i < to) read_item<S>(ops, f[1 + i / NF], i % NF, a, b, 1 + i / NF);
  };
  constexpr int N0 = NF + HEAD, N1 = 2 * NF - HEAD, M1 = S::FM / 2;
  phase<FIRST, S>(f[0], acc, [&](int m) { early(m * N0 / S::FM, (m + 1) * N0 / S::FM); }, none);
  phase<false, S>(f[1], acc, [&](int m) { early(N0 + (m < M1 ? m * N1 / M1 : N1), N0 + (m + 1 < M1 ? (m + 1) * N1 / M1 : N1)); }, none);
  // every wavefront holds all of the stage's fragments: its slot is free (and with three slots the next stage has landed)
  if (S::SLOTS > 2) {
    constexpr int N = (S::SLOTS - 2) * S::NL + STORES;
    wait_loads<(N < 63 ? N : 63)>();
  }
  __syncthreads();
  auto refill = [&](int from, int to) {
#pragma unroll
    for (int I = 0; I < S::NL; ++I)
      if (I >= from && I < to) ops.load(ops.nth(I), fill_a, fill_b);
  };
  constexpr int L0 = S::NL / 2, L1 = S::NL - L0;
  phase<false, S>(f[2], acc, none, [&](int m) { if (FILL) refill(m * L0 / S::FM, (m + 1) * L0 / S::FM); });
  if (S::SLOTS == 2) {   // the next stage has landed
    constexpr int N = L0 + STORES;
    wait_loads<(N < 63 ? N : 63)>();
    __syncthreads();
  }
  phase<false, S>(f[3], acc,
                  [&](int m) {
#pragma unroll
                    for (int i = 0; i < NF; ++i)
                      if (i >= m * NF / M1 && i < (m + 1 < M1 ? (m + 1) * NF / M1 : NF)) read_item<S>(ops, f[0], i, an, bn, 0);
                  },
                  [&](int m) { if (FILL) refill(L0 + m * L1 / S::FM, L0 + (m + 1) * L1 / S::FM); });
}

// ======================================================================================
// scatter2scatter
// ======================================================================================
// How the tiles of a launch are dealt to the G blocks.  Tiles are numbered densely (tile_coords); full rounds deal G tiles.
// The `rest` < G tiles left would keep few compute units busy for a whole tile: their contraction is cut into `split` chunks of
// `chunk` stages for the blocks still free; the chunks leave fp32 partial tiles that a second kernel adds in chunk order
// (deterministic) and stores.
struct TilePlan {
  int m_tiles, rounds, rest, split, chunk;
};
// first[e] = M-tiles of the experts before e, by every wavefront for itself (all write the same); returns first[E].  A tile's expert is
// then found by one comparison per lane, where a search that adds up the experts' tiles again is a chain of ten lane exchanges, which
// the matrix cores wait for at every tile.
template <typename S> __device__ __forceinline__ int number_tiles(const int32_t *offsets, int E, int *first, int lane) {
  int base = 0;
  if (lane == 0) first[0] = 0;
  for (int c0 = 0; c0 < E; c0 += 64) {
    const int x = c0 + lane;
    int n = x < E ? (offsets[x + 1] - offsets[x] + S::TM - 1) / S::TM : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(n, d, 64);
      if (lane >= d) n += up;
    }
    if (x < E) first[x + 1] = base + n;
    base += __builtin_amdgcn_readlane(n, 63);
  }
  return base;
}
template <typename S>
__device__ __forceinline__ void find_tile(const int32_t *offsets, const int *first, int E, int tile, int lane, int &e, int &row0, int &row_end) {
  e = E - 1;
  for (int c0 = 0; c0 < E; c0 += 64) {
    const unsigned long long owns = __ballot(first[min(c0 + lane, E - 1) + 1] > tile);
    if (!owns) continue;
    e = c0 + __ffsll((long long)owns) - 1;
    break;
  }
  row0 = __builtin_amdgcn_readfirstlane(offsets[e]) + (tile - __builtin_amdgcn_readfirstlane(first[e])) * S::TM;
  row_end = __builtin_amdgcn_readfirstlane(offsets[e + 1]);
}
template <typename S>
__device__ __forceinline__ TilePlan plan_tiles(int m_tiles, int tiles_n, int ns, int G, bool static2, bool may_split) {
  TilePlan p;
  p.m_tiles = m_tiles;
  const long long total = (long long)p.m_tiles * tiles_n;
  p.rounds = (int)(total / G);
  p.rest = (int)(total - (long long)p.rounds * G);
  p.split = 1;
  p.chunk = ns;
  if (may_split && p.rest > 0) p.split = choose_split(ns, G / p.rest, static2, p.chunk);
  return p;
}

// Sources of the loader's current tile: range-checked windows, and per-lane 32-bit byte offsets at contraction offset 0.
template <typename S, bool TRANS_W, bool KTAIL, bool SWIGLU> struct S2SOps {
  int32x4 win_a, win_b;
  uint32_t oa[S::NLA], ob[2];        // ob: even and odd load instructions; a pair of them lies b_rows bytes behind the one before
  uint32_t ta[2], tb[2];             // KTAIL, even and odd instructions: all ones where the lane's chunk of the last stage lies past K
  uint32_t b_step, b_rows;           // bytes the W source moves per stage, and per pair of load instructions
  uint32_t fa[4], fb[4];             // the lane's fragments inside a slot: by sixteenth of the contraction, or (W as stored) by column fragment
  int step, last;                    // stage the next loads fetch; the contraction's last stage
  int uwave;
  int again;                         // S::ONCE: above 0 where the expert has further tiles, which read the same weights
  // The order of a stage's load instructions: A and W in turn; with SwiGLU, whose tiles take W's columns from two places, A first (not
  // in HalfShort, whose launches wait for W: 16 experts of 62 rows, 4096 -> 2 x 512, 61 -> 59.5 us).
  __device__ static constexpr int nth(int i) {
    if (SWIGLU && (S::NLA == S::NLB || S::SLOTS > 2)) return i;
    if (S::NLA == S::NLB) return i & 1 ? S::NLA + i / 2 : i / 2;
    return i % 3 ? S::NLA + i / 3 * 2 + i % 3 - 1 : i / 3;
  }
  __device__ __forceinline__ void load(int I, uint32_t fill_a, uint32_t fill_b) const {
    if (I < S::NLA) {
      uint32_t off = oa[I] + (uint32_t)step * (SK * 2);
      if (KTAIL) off |= step == last ? ta[I & 1] : 0u;
      load16_to_lds_checked(win_a, off, fill_a + uwave * (S::NLA * 1024), I * 1024);
    } else {
      const int J = I - S::NLA;
      uint32_t off = ob[J & 1] + ((uint32_t)(J >> 1) * b_rows + (uint32_t)step * b_step);
      if (KTAIL && TRANS_W) off |= step == last ? tb[J & 1] : 0u;
      const uint32_t lds = fill_b + uwave * (S::NLB * 1024);
      if (S::ONCE) load16_to_lds_checked_or_once(win_b, off, lds + J * 1024, again);
      else load16_to_lds_checked(win_b, off, lds, J * 1024);
    }
  }
  __device__ __forceinline__ bf16x8 frag_a(const char *slot, int i, int kk) const { return line_frag(slot + fa[kk], i); }
  __device__ __forceinline__ bf16x8 frag_b(const char *slot, int j, int kk) const {
    return TRANS_W ? line_frag(slot + fb[kk], j) : rows_frag(slot + fb[j], kk);
  }
};

// ACT 1: fused SwiGLU keeping the pre-activation, 2: without, 3: fused SwiGLU derivative and dp (the W2^T input-gradient
// product of Alg. 3's backward, see store_wave_tile_swiglu_bwd), 4: dp from the saved H in that product's epilogue for any
// activation (store_wave_tile_dp), 5: 4 with the routing-weighted hidden rows written as well, 6: 5 with H and dH in slot order, 7: 3 with the routing-weighted hidden
// rows written as well.
// STATIC2 (Big only): the contraction is an even number of whole stages, so every tile starts in LDS slot 0 and the loop is written
// out two stages at a time with the slot as a compile-time constant: all LDS addresses become a loop-invariant register plus an
// immediate.  Without it the contraction may be any multiple of 8 (KTAIL masks the last stage).
// WIDE: a scattered output of 4 GB or more.
template <typename S, bool TRANS_W, bool SCATTER_OUT, int ACT, bool STATIC2, bool WIDE>
__global__ void __launch_bounds__(NTHREADS, 1) s2s_stream_kernel(S2SArgs a, int tiles_n, int group_m, uint32_t magic_a) {
  constexpr bool SWIGLU = ACT == 1 || ACT == 2;
  constexpr bool GATE_UP = ACT == 3 || ACT == 7;
  constexpr bool KTAIL = !STATIC2;
  constexpr bool DENSE_PAIR = ACT == 0 && !SCATTER_OUT;   // S2SArgs::C2 may be set
  constexpr int STORES = EpilogueStores<S::FM, ACT>;
  static_assert(!SWIGLU || (!TRANS_W && !SCATTER_OUT), "the fused activation belongs to the forward, sorted-output product");
  static_assert(ACT < 3 || (TRANS_W && SCATTER_OUT == (ACT == 6)), "the fused derivative belongs to the W^T product");
  static_assert(!STATIC2 || S::SLOTS == 2, "the unrolled loop walks two slots");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int s_off[MAX_E + 1], s_first[MAX_E + 1];
  // Order indices of the rows of up to four open tiles.  With the shortest contraction the kernel takes (two stages) the
  // loader has opened tile n+2 and requested the rows of tile n+3 while tile n's epilogue still reads its destination
  // rows, so four entries are live at once.
  __shared__ int s_idx[4][S::TM];
  // The open tiles themselves, left by the loader's search for the multiplying side.  One ring for the block: every wavefront writes the
  // same values and may read what another wrote.  What keeps an entry until the slowest has read it is the barriers of each stage: with
  // two stages or more per tile no wavefront has opened a tile past n + 3 while another still fetches the entry of n + 1.
  __shared__ __attribute__((aligned(16))) int s_tile[4][4];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int uwm = uwave >> 1, uwn = uwave & 1;
  const int G = gridDim.x;
  const int pos = ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3);   // blocks b, b + 8, ... share an XCD and get consecutive tiles
  const int ns = (a.K + SK - 1) / SK;

  const bool probe = a.clock_probe && blockIdx.x < MAX_STREAM_GRID;
  const unsigned long long probe_c0 = probe ? clock64() : 0ull, probe_t0 = probe ? wall_clock64() : 0ull;
  for (int i = threadIdx.x; i <= a.E; i += NTHREADS) s_off[i] = a.offsets ? a.offsets[i] : a.Tk / a.E * i;
  __syncthreads();

  const TilePlan plan = plan_tiles<S>(number_tiles<S>(s_off, a.E, s_first, lane), tiles_n, ns, G, STATIC2, ACT == 0 && a.tail_ws != nullptr);
  // This block's part of the last, partial round: tile number (-1: none), chunk of its contraction, index of the fp32
  // partial tile it leaves (-1: the tile is whole).
  int last_tile = -1, last_h0 = 0, last_hn = ns, last_part = -1;
  if (pos < plan.rest * plan.split) {
    const int chunk = pos % plan.split;
    last_tile = plan.rounds * G + pos / plan.split;
    if (plan.split > 1) {
      last_h0 = chunk * plan.chunk;
      last_hn = min(ns, last_h0 + plan.chunk) - last_h0;
      last_part = pos;
    }
  }
  const int rounds = plan.rounds, m_tiles = plan.m_tiles;
  // Arguments needed once per tile are read from the kernel's argument segment again where they are used: kept in scalar
  // registers they would not fit beside the loader's state, and the loop would fetch spilled registers every stage.
  auto args = [&]() {
    auto p = (const __attribute__((address_space(4))) S2SArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(p));
    return p;
  };
  struct Tile {
    int seq;                    // position in this block's tile list (-1 before the first)
    int e, row0, row_end, n0;
  };
  // next tile (or chunk of a tile of the last round) of this block after t
  auto next_tile = [&](Tile &t) -> bool {
    const int seq = t.seq + 1;
    if (seq > rounds || (seq == rounds && last_tile < 0)) return false;
    const int w = seq < rounds ? seq * G + pos : last_tile;
    int mt, nt;
    tile_coords(w, m_tiles, tiles_n, group_m, mt, nt);
    t.seq = seq;
    find_tile<S>(s_off, s_first, a.E, mt, lane, t.e, t.row0, t.row_end);
    t.n0 = nt * (SWIGLU ? TB / 2 : TB);   // SwiGLU tiles hold 128 gate columns and the 128 up columns pairing with them
    *reinterpret_cast<int4 *>(s_tile[seq & 3]) = make_int4(t.e, t.row0, t.row_end, t.n0);
    return true;
  };
  // the multiplying side's next tile, which the loader has opened before
  const int tiles = rounds + (last_tile >= 0 ? 1 : 0);
  auto follow = [&](Tile &t) -> bool {
    if (t.seq + 1 >= tiles) return false;
    ++t.seq;
    const int4 v = *reinterpret_cast<const int4 *>(s_tile[t.seq & 3]);
    t.e = __builtin_amdgcn_readfirstlane(v.x);
    t.row0 = __builtin_amdgcn_readfirstlane(v.y);
    t.row_end = __builtin_amdgcn_readfirstlane(v.z);
    t.n0 = __builtin_amdgcn_readfirstlane(v.w);
    return true;
  };
  auto stages = [&](const Tile &t) { return t.seq < rounds ? ns : last_hn; };
  auto first_step = [&](const Tile &t) { return t.seq < rounds ? 0 : last_h0; };
  // order indices of a tile's rows -> s_idx[seq & 3] (rows past the segment repeat its last row); with 128 rows
  // wavefronts 2 and 3 load the same again, so that every wavefront counts the same loads
  auto fetch_rows = [&](const Tile &t) {
    const auto p = args();
    const int32_t *o = p->a_map.o ? p->a_map.o : p->c_map.o;   // both maps use the same order indices
    if (!o) return;
    const int part = wave & (S::TM / 64 - 1);
    const int i = min(t.row0 + part * 64 + lane, t.row_end - 1);
    load4_to_lds(o + i, __builtin_amdgcn_readfirstlane(lds_address((const char *)&s_idx[t.seq & 3][0])) + (uwave & (S::TM / 64 - 1)) * 256);
  };

  S2SOps<S, TRANS_W, KTAIL, SWIGLU> ops;
  ops.uwave = uwave;
  ops.b_step = TRANS_W ? (uint32_t)(SK * 2) : (uint32_t)(SK * 2) * (uint32_t)a.ldw;
  ops.b_rows = (TRANS_W ? 32u : 8u) * (uint32_t)a.ldw;
  ops.last = ns - 1;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ops.fa[q] = line_frag_offset(wm * (S::TM / 2), q, lane);
    ops.fb[q] = TRANS_W ? line_frag_offset(wn * (TB / 2), q, lane) : rows_frag_offset(wn * (TB / 2) + q * 32, lane);
  }
  uint32_t chunk[2];                 // source chunk of the lane's 16 bytes in a row of 128, even and odd load instructions
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    chunk[p] = (uint32_t)((lane & 7) ^ line_swz(p * 8 + (lane >> 3)));
    ops.ta[p] = ops.tb[p] = KTAIL && (ns - 1) * SK + (int)chunk[p] * 8 >= a.K ? ~0u : 0u;
  }
  // order index -> source row, with no branch for fan-out 1
  const uint32_t whole = magic_a ? 0u : ~0u;
  auto source_row = [&](uint32_t slot) { return __umulhi(slot, magic_a) + (slot & whole); };
  auto setup_sources = [&](const Tile &t) {
    const auto p = args();
    const int K = p->K, N = p->N;
    const uint32_t row_bytes = (uint32_t)K * 2u, ldw_bytes = (uint32_t)p->ldw * 2u;
    const bool gathered = p->a_map.o != nullptr;
    // gathered rows are addressed from the start of A, expert-sorted rows from the tile's first row
    const bool second = DENSE_PAIR && p->C2 && t.e == 1;
    ops.win_a = buffer_window((const bf16_t *)(second ? p->A2 : p->A) + (gathered ? 0 : (size_t)t.row0 * K),
                              (gathered ? source_row((uint32_t)p->Tk) : (uint32_t)min(S::TM, t.row_end - t.row0)) * row_bytes);
    ops.win_b = buffer_window((const bf16_t *)(second ? p->W2 : p->W) + (size_t)t.e * p->w_stride, (uint32_t)(TRANS_W ? N : K) * ldw_bytes);
    if (S::ONCE) ops.again = t.row_end - __builtin_amdgcn_readfirstlane(s_off[t.e]) - S::TM;
    const int *idx = &s_idx[t.seq & 3][0];
    // Rows past the segment read zeros: an offset that stays past the window at every stage.  (Repeating the segment's last row, as the
    // order indices there do, is as right, but its products cost the power of real ones.)
    const uint32_t past = 0u - row_bytes - SK * 2u;
#pragma unroll
    for (int I = 0; I < S::NLA; ++I) {
      const int r = (wave * S::NLA + I) * 8 + (lane >> 3);
      uint32_t src = (uint32_t)r;
      if (gathered) src = source_row((uint32_t)idx[r]);
      ops.oa[I] = r < t.row_end - t.row0 ? src * row_bytes + chunk[I & 1] * 16u : past;
    }
    // Rows (W^T) or columns past N read what lies there or zeros; they end up in outputs that are never stored.
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      if (TRANS_W) {
        ops.ob[p] = (uint32_t)(t.n0 + wave * 64 + p * 8 + (lane >> 3)) * ldw_bytes + chunk[p] * 16u;
      } else {
        const int r = wave * 16 + p * 2 + (lane >> 5), c = (lane & 31) ^ tr_swz(r);
        int col = t.n0 + c * 8;
        if (SWIGLU) {
          // tile column v = c * 8: wavefront column half v / 128 takes 64 gate columns then their 64 up columns
          const int v = c * 8, w = v & 127, gate = t.n0 + (v >> 7) * 64 + (w & 63);
          col = (gate < N / 2) ? gate + (w >> 6) * (N / 2) : N;
        }
        if (col >= N) col = 0;
        ops.ob[p] = (uint32_t)r * ldw_bytes + (uint32_t)col * 2u;
      }
    }
  };

  // ---- open the first two tiles
  Tile lt{-1, 0, 0, 0, 0};
  if (!next_tile(lt)) return;
  Tile ct = lt;                // the multiplying side starts on the same tile
  Tile upcoming = lt;          // tile the loader will open next
  bool have_upcoming = next_tile(upcoming);
  fetch_rows(lt);
  if (have_upcoming) fetch_rows(upcoming);
  wait_loads<0>();
  __syncthreads();
  setup_sources(lt);
  ops.step = first_step(lt);
  int step_end = ops.step + stages(lt);
  bool loader_live = true;
  // loader moves one stage on; at a tile end it opens the upcoming tile and requests the rows of the one after
  auto advance_loader = [&]() {
    if (!loader_live) return;
    if (++ops.step < step_end) return;
    if (!have_upcoming) {
      loader_live = false;
      --ops.step;              // stages past the end repeat the last one's addresses
      return;
    }
    lt = upcoming;
    ops.step = first_step(lt);
    step_end = ops.step + stages(lt);
    have_upcoming = next_tile(upcoming);
    if (have_upcoming) fetch_rows(upcoming);
    setup_sources(lt);
  };

  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
#pragma unroll 1
  for (int st = 0; st < S::SLOTS; ++st) {
#pragma unroll
    for (int I = 0; I < S::NL; ++I) ops.load(I, lds0 + st * S::A_BYTES, lds0 + S::SLOTS * S::A_BYTES + st * B_BYTES);
    advance_loader();
  }
  wait_loads<(S::SLOTS - 1) * S::NL>();   // the first stage has landed
  __syncthreads();
  f32x16 acc[S::FM][FR];
  Frags<S> f[4];
#pragma unroll
  for (int i = 0; i < S::NF; ++i) read_item<S>(ops, f[0], i, smem, smem + S::SLOTS * S::A_BYTES, 0);

  int cur = 0;                 // LDS slot of the stage at hand (0 at every tile start with STATIC2)
  auto next_slot = [&](int slot) { return slot == S::SLOTS - 1 ? 0 : slot + 1; };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  for (;;) {   // one tile per trip
    const int hn = stages(ct);
    // the stores of the previous tile's epilogue lie behind the loads that the first stage's wait is for
    if constexpr (STATIC2) {
      if (ct.seq > 0) stage_step<true, false, STORES, S>(ops, f, acc, smem, lds0, I0{}, I1{});
      else stage_step<true, false, 0, S>(ops, f, acc, smem, lds0, I0{}, I1{});
      advance_loader();
      stage_step<false, false, 0, S>(ops, f, acc, smem, lds0, I1{}, I0{});
      advance_loader();
      for (int h = 2; h < hn; h += 2) {
        stage_step<false, false, 0, S>(ops, f, acc, smem, lds0, I0{}, I1{});
        advance_loader();
        stage_step<false, false, 0, S>(ops, f, acc, smem, lds0, I1{}, I0{});
        advance_loader();
      }
    } else {
      if (ct.seq > 0) stage_step<true, false, STORES, S>(ops, f, acc, smem, lds0, cur, next_slot(cur));
      else stage_step<true, false, 0, S>(ops, f, acc, smem, lds0, cur, next_slot(cur));
      advance_loader();
      cur = next_slot(cur);
      for (int h = 1; h < hn - 1; ++h) {
        stage_step<false, false, 0, S>(ops, f, acc, smem, lds0, cur, next_slot(cur));
        advance_loader();
        cur = next_slot(cur);
      }
      stage_step<false, true, 0, S>(ops, f, acc, smem, lds0, cur, next_slot(cur));
      if (!S::PATCH_IN_SLOT) advance_loader();
    }
    const int lane = ACT == 6 ? lane_here(threadIdx.x & 63) : (int)(threadIdx.x & 63);
    char *patch = S::PATCH_IN_SLOT ? smem + S::SLOTS * S::A_BYTES + cur * B_BYTES + uwave * (S::NLB * 1024)
                                   : smem + S::RING_BYTES + uwave * EPI_WAVE_BYTES;
    const auto p = args();
    const int N = p->N;
    const int rbase = ct.row0 + uwm * (S::TM / 2);            // the wavefront's first row
    const int left = max(min(S::TM / 2, ct.row_end - rbase), 0);
    // a 64-column block of an expert-sorted tensor with `ld` columns: `col` its first column, `room` how many exist from there on
    auto sorted_window = [&](const void *base, int ld, int elem) {
      return make_window((const char *)base + (size_t)rbase * ld * elem, (uint32_t)left * (uint32_t)ld * (uint32_t)elem);
    };
    auto sorted_block = [&](window_t win, int ld, int fm, int col, int room) {
      BlockDest d{win, {}};
      const uint32_t mine = (lane & 7) * 8 < room ? (uint32_t)(lane >> 3) * (uint32_t)ld * 2u + (uint32_t)(col + (lane & 7) * 8) * 2u : OFF_WINDOW;
#pragma unroll
      for (int it = 0; it < 4; ++it) d.off[it] = mine + (uint32_t)(fm * 32 + it * 8) * (uint32_t)ld * 2u;
      return d;
    };
    // the same of a tensor in slot order: the rows' places come from the order indices
    auto slot_block = [&](window_t win, int n, const int *places, int rows, int fm, int col0) {
      BlockDest d{win, {}};
      const int col = col0 + (lane & 7) * 8;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = fm * 32 + it * 8 + (lane >> 3);
        const uint32_t off = (uint32_t)places[r] * ((uint32_t)n * 2u) + (uint32_t)col * 2u;
        d.off[it] = r < rows && col < n ? off : ~0u;
      }
      return d;
    };
    if constexpr (SWIGLU) {
      const int half_n = N / 2, gcol = ct.n0 + uwn * (TB / 4);
      const window_t win_h = sorted_window(p->H, half_n, 2);
      const window_t win_p = ACT == 1 ? sorted_window(p->C, N, 2) : win_h;
      store_wave_tile_swiglu<ACT == 1>(
          acc, patch, [&](int fm, int half) { return sorted_block(win_p, N, fm, half * half_n + gcol, half_n - gcol); },
          [&](int fm) { return sorted_block(win_h, half_n, fm, gcol, half_n - gcol); }, lane);
    } else if constexpr (ACT >= 3) {
      const int gcol = ct.n0 + uwn * (TB / 2), ldc = GATE_UP ? 2 * N : N;
      const uint32_t slot_bytes = (uint32_t)p->Tk * (uint32_t)N * 2u;                 // ACT 6: of dH and of H
      const window_t win_c = ACT == 6 ? make_window(p->C, slot_bytes) : sorted_window(p->C, ldc, 2);
      BwdRows b;
      b.saved = ACT == 6 ? make_window(p->H_in, slot_bytes) : sorted_window(GATE_UP ? p->Hpre_in : p->H_in, ldc, 2);
      b.places = &s_idx[ct.seq & 3][uwm * (S::TM / 2)];
      b.left = left;
      b.saved_bytes = (uint32_t)ldc * 2u;
      if (ACT == 7) b.hidden = sorted_window(p->H_in, N, 2);
      b.scale = make_window(p->row_scale, (uint32_t)p->Tk * 4u);
      b.dp = sorted_window(p->dp_part, 2 * tiles_n, 4);
      b.part_bytes = (uint32_t)tiles_n * 8u;
      b.part_col = (uint32_t)(ct.n0 / TB) * 2u + uwn;
      b.n = N;
      b.gcol = gcol;
      const window_t win_w = ACT >= 5 ? sorted_window(p->Hw_out, N, 2) : win_c;
      auto dest_hw = [&](int fm, int half) { return sorted_block(win_w, N, fm, gcol + half * 64, N - gcol - half * 64); };
      if constexpr (GATE_UP) {
        store_wave_tile_swiglu_bwd<ACT == 7>(
            acc, patch, b,
            [&](int fm, int half, int up) { return sorted_block(win_c, ldc, fm, up * N + gcol + half * 64, N - gcol - half * 64); }, dest_hw, lane);
      } else {
        auto dest = [&](int fm, int half) {
          if constexpr (ACT == 6) return slot_block(win_c, N, b.places, left, fm, gcol + half * 64);
          else return sorted_block(win_c, ldc, fm, gcol + half * 64, N - gcol - half * 64);
        };
        store_wave_tile_dp<ACT >= 5, ACT == 6>(acc, patch, b, dest, dest_hw, lane);
      }
    } else {
      const int wcol = ct.n0 + uwn * (TB / 2);
      const int *idx = &s_idx[ct.seq & 3][uwm * (S::TM / 2)];
      if (ct.seq == rounds && last_part >= 0) {
        store_wave_partial(acc, p->tail_ws + (size_t)last_part * S::PART + (size_t)(uwm * (S::TM / 2)) * TB + uwn * (TB / 2), lane);
      } else if constexpr (SCATTER_OUT && WIDE) {
        bf16_t *C = (bf16_t *)p->C;
        store_wave_tile(acc, patch, [&](int fm, int half) {
          WideBlockDest d;
          const int col = wcol + half * 64 + (lane & 7) * 8;
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            const int r = fm * 32 + it * 8 + (lane >> 3);
            d.p[it] = r < left && col < N ? C + (size_t)idx[r] * N + col : (bf16_t *)g_trash + lane * 8;
          }
          return d;
        }, lane);
      } else if constexpr (SCATTER_OUT) {
        const window_t win = make_window(p->C, (uint32_t)p->Tk * (uint32_t)N * 2u);
        store_wave_tile(acc, patch, [&](int fm, int half) { return slot_block(win, N, idx, left, fm, wcol + half * 64); }, lane);
      } else {
        const window_t win = sorted_window(p->C2 && ct.e == 1 ? p->C2 : p->C, N, 2);
        store_wave_tile(acc, patch, [&](int fm, int half) { return sorted_block(win, N, fm, wcol + half * 64, N - wcol - half * 64); },
                        lane);
      }
    }
    if constexpr (S::PATCH_IN_SLOT) {   // the refill that the last stage held back
#pragma unroll
      for (int I = 0; I < S::NL; ++I) ops.load(I, lds0 + cur * S::A_BYTES, lds0 + S::SLOTS * S::A_BYTES + cur * B_BYTES);
      advance_loader();
    }
    if constexpr (!STATIC2) cur = next_slot(cur);
    if (!follow(ct)) break;
  }
  wait_loads<0>();
  if (probe && threadIdx.x == 0) {
    unsigned long long *report = args()->clock_probe;
    report[2 * blockIdx.x] = clock64() - probe_c0;
    report[2 * blockIdx.x + 1] = wall_clock64() - probe_t0;
  }
}

// Second pass of a split last round: adds the chunks' fp32 partial tiles in chunk order, rounds once and stores the rows where the
// unsplit epilogue would have (expert-sorted or scattered).  The plan is recomputed from the same inputs as in the main kernel.
// How many tiles are left over only the device knows, so a fixed number of blocks deals itself the TAIL_SLICES slices of however
// many there are: latency of each thread's chain of loads bounds it, not bandwidth, so a tile is spread over many threads, but a
// block for every slice of every tile that could be left (8192, most of which rebuilt the plan and left) took 16 us for the 16 tiles
// of an 8192 x 1024 output, 12 for those of 6002 x 1280 and 7 where nothing was left; TAIL_BLOCKS blocks take 6, 5 and 5.
constexpr int TAIL_SLICES = 32, TAIL_BLOCKS = 1024;
template <typename S, bool SCATTER_OUT>
__global__ void __launch_bounds__(256) s2s_tail_reduce_kernel(S2SArgs a, int tiles_n, int group_m, int G, int static2) {
  __shared__ int s_off[MAX_E + 1], s_first[MAX_E + 1];
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i <= a.E; i += 256) s_off[i] = a.offsets ? a.offsets[i] : a.Tk / a.E * i;
  __syncthreads();
  const TilePlan plan = plan_tiles<S>(number_tiles<S>(s_off, a.E, s_first, lane), tiles_n, (a.K + SK - 1) / SK, G, static2 != 0, true);
  if (plan.split <= 1) return;
  constexpr int PER_SLICE = S::PART / 4 / TAIL_SLICES;
  for (int unit = blockIdx.x; unit < plan.rest * TAIL_SLICES; unit += TAIL_BLOCKS) {
    const int tile = unit / TAIL_SLICES, slice = unit % TAIL_SLICES;
    int mt, nt, e, row0, row_end;
    tile_coords(plan.rounds * G + tile, plan.m_tiles, tiles_n, group_m, mt, nt);
    find_tile<S>(s_off, s_first, a.E, mt, lane, e, row0, row_end);
    const int n0 = nt * TB;
    const float *part = a.tail_ws + (size_t)tile * plan.split * S::PART;
    bf16_t *C = (bf16_t *)(!SCATTER_OUT && a.C2 && e == 1 ? a.C2 : a.C);
    for (int i = slice * PER_SLICE + threadIdx.x; i < (slice + 1) * PER_SLICE; i += 256) {
      const int row = row0 + (i * 4) / TB, col = n0 + (i * 4) % TB;
      if (row >= row_end || col >= a.N) continue;
      const int dst = SCATTER_OUT ? a.c_map.o[row] : row;
      float4 v[MAX_SPLIT];                      // all chunks in flight before the first is added
#pragma unroll
      for (int c = 0; c < MAX_SPLIT; ++c)
        v[c] = c < plan.split ? reinterpret_cast<const float4 *>(part + (size_t)c * S::PART)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int c = 1; c < MAX_SPLIT; ++c) { v[0].x += v[c].x; v[0].y += v[c].y; v[0].z += v[c].z; v[0].w += v[c].w; }
      bf16x4 o;
      o[0] = (bf16_t)v[0].x; o[1] = (bf16_t)v[0].y; o[2] = (bf16_t)v[0].z; o[3] = (bf16_t)v[0].w;
      *reinterpret_cast<bf16x4 *>(C + (size_t)dst * a.N + col) = o;
    }
  }
}

// ======================================================================================
// groupXTY, persistent: dW[e] = Xbar_e^T dYbar_e over the rows of each expert's segment.  An operand lies expert-sorted, or
// (DWArgs' row maps) its rows are read from their source through the order indices, with no sorted copy.
// ======================================================================================
// The loader's cursor runs two stages (three where it fetches order indices) ahead of the multiplying side over the same sequence: the
// stages (of 64 rows) of a tile rounded up to an even number (at least two), tiles in largest-expert-first order.  Rows past a segment's
// end load zeros, so a tile of an empty expert multiplies zeros and writes zeros.  One wavefront per SIMD: what a stage's bookkeeping
// takes the matrix cores wait for, so everything that is constant over a tile is worked out once per tile, and a step to the next
// stage is a few scalar additions.
struct DWCursor {
  int seq;               // position in this block's tile list
  int step, ns;          // stage within the tile, stages of the tile
  int left;              // rows of the segment from the stage's first on (0 or less: none)
  int e, m0, n0;
  bool further;          // a tile of dW3
  const char *pa, *pb;   // the stage's first row of each operand; the start of a source whose rows are read through the order indices
  uint32_t sa, sb;       // bytes from one stage to the next (0 for such a source)
  const int32_t *po;     // order indices from the stage's first row on
};
struct DWTile {          // the multiplying side's tile
  int seq, e, m0, n0, ns;
  bool further;
};

// How the operands of a launch lie (kernels of their own: the choice sits in every load): DW_ONE sorted; DW_A, DW_B, DW_AB the rows of
// A, of B or of both read through the order indices; DW_PAIR sorted, segment 1 is the second weight gradient of DWArgs; DW_TWO every
// expert's tiles are followed by those of its dW3, whose A3, like the first one's B, may be read through the order indices.
enum { DW_ONE, DW_A, DW_B, DW_AB, DW_PAIR, DW_TWO };

template <int KIND> struct DWStreamOps {
  static constexpr bool ROWS_A = KIND == DW_A || KIND == DW_AB || KIND == DW_TWO, ROWS_B = KIND == DW_B || KIND == DW_AB || KIND == DW_TWO;
  int uwave;
  // The loader's current stage: range-checked windows that start at its first row and end with its rows of the expert's segment (rows
  // past it, padded stages and empty experts read zeros and add nothing to the sum), and per-lane byte offsets of the tile's columns for
  // even and odd load instructions; a pair of them (four rows) lies pair_a or pair_b bytes behind the one before.
  int32x4 win_a, win_b;
  uint32_t oa[2], ob[2], pair_a, pair_b;
  uint32_t fa[4], fb[4];     // the lane's column fragments inside a slot
  // Rows read through the order indices: the stage's indices of the lane's rows, by load instruction; bytes per source row (0: the
  // operand lies sorted); multiply-high that divides twice an index by twice the fan-out; rows of the segment from the stage's first
  // on, and the lane's first row.  Lanes past the segment read zeros by an offset outside the window.
  uint32_t order[Big::NLA];
  uint32_t mul_a, mul_b, magic_a, magic_b;
  int left, row;
  __device__ __forceinline__ uint32_t through(int I, uint32_t off, uint32_t mul, uint32_t magic) const {
    off += __umul24(__umulhi(order[I] * 2u, magic), mul);
    return row + 2 * I < left ? off : ~0u;
  }
  __device__ static constexpr int nth(int i) { return i & 1 ? Big::NLA + i / 2 : i / 2; }
  __device__ __forceinline__ void load(int I, uint32_t fill_a, uint32_t fill_b) const {
    if (I < Big::NLA) {
      uint32_t off = oa[I & 1] + (uint32_t)(I >> 1) * pair_a;
      if (ROWS_A) off = through(I, off, mul_a, magic_a);
      load16_to_lds_checked(win_a, off, fill_a + uwave * (Big::NLA * 1024), I * 1024);
    } else {
      const int J = I - Big::NLA;
      uint32_t off = ob[J & 1] + (uint32_t)(J >> 1) * pair_b;
      if (ROWS_B) off = through(J, off, mul_b, magic_b);
      load16_to_lds_checked(win_b, off, fill_b + uwave * (Big::NLB * 1024), J * 1024);
    }
  }
  __device__ __forceinline__ bf16x8 frag_a(const char *slot, int i, int kk) const { return rows_frag(slot + fa[i], kk); }
  __device__ __forceinline__ bf16x8 frag_b(const char *slot, int j, int kk) const { return rows_frag(slot + fb[j], kk); }
};

constexpr uint32_t MAX_SOURCE_BYTES = 0xfffffff0u;      // window of rows read through the order indices

// tile number inside an expert -> first row and column of the tile: bands of group_m M-tiles, N-tile by
// N-tile, so that the 32 consecutive tiles an XCD holds at a time form a compact patch sharing few panels
__device__ __forceinline__ void dw_tile_origin(int t, int tiles_m, int tiles_n, int &m0, int &n0) {
  const int group_m = (tiles_m % 8 == 0) ? 8 : ((tiles_m % 4 == 0) ? 4 : ((tiles_m % 2 == 0) ? 2 : 1));
  const int band = t / (group_m * tiles_n), r = t - band * (group_m * tiles_n);
  m0 = (band * group_m + r % group_m) * TB;
  n0 = (r / group_m) * TB;
}
// rows of chunk `chunk` of `split` of the segment [lo, hi): chunks are whole pairs of stages
__device__ __forceinline__ void dw_chunk_rows(int lo, int hi, int split, int chunk, int &clo, int &chi) {
  const int nh = (hi - lo + HK - 1) / HK;
  const int len = (((nh + split - 1) / split + 3) & ~3) * HK;
  clo = min(hi, lo + chunk * len);
  chi = min(hi, clo + len);
}

// split > 1 (only when all experts' tiles times split fit one round of the grid): unit T is chunk T % split of
// tile T / split, experts in their own order, and the result is an fp32 partial tile number T in a.split_ws.
//
// A sorted copy of the rows costs a pass over them that writes [Tk, width] and a launch, and the product reads that copy instead of a
// source that is fan-out times smaller.  Training steps with the copies / with rows through the order indices, interleaved on one box,
// in us: granular layer (8192 tokens, 64 experts, k = 8, 2048 -> 2 x 512) 1605 / 1544, one ParallelLinear (16396 rows, 2048 -> 1536) 408 /
// 393, attention layer (8192 tokens, k = 4) 1443 / 1382, small layer (8192 rows, 1024 -> 2 x 2816) 610 / 605, its weight gradients 69 + 113.
// With the tile's constants worked out in every stage instead of once per tile the same launches gained less: 1567 of 1648 where these take
// 1544 of 1605, and the small layer lost 1 %.
//
// Rows through the order indices (ROWS): a wavefront needs the indices of the 16 rows of a stage that it loads itself.  It fetches them
// into LDS by a load of its own, issued a stage before the operand loads that use them: that stage's wait covers it, so the
// fetch adds no wait and no barrier, and an index becomes an offset in the shadow of the matrix instructions.
template <int KIND> __global__ void __launch_bounds__(NTHREADS, 1) dw_stream_kernel(DWArgs a, int tiles_m, int tiles_n, int split, uint32_t magic_a, uint32_t magic_b) {
  constexpr bool DENSE_PAIR = KIND == DW_PAIR, ROWS = DWStreamOps<KIND>::ROWS_A || DWStreamOps<KIND>::ROWS_B;
  __shared__ __attribute__((aligned(16))) uint32_t s_rows[ROWS ? 2 : 1][ROWS ? 4 : 1][64];   // by stage parity and wavefront
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int s_off[MAX_E + 1];
  __shared__ int s_order[MAX_E];      // experts, largest segment first

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int uwm = __builtin_amdgcn_readfirstlane(wm), uwn = __builtin_amdgcn_readfirstlane(wn);
  const int G = gridDim.x;
  const int slot_in_round = ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3);  // XCD-contiguous tiles
  const int tiles_m3 = (a.M3 + TB - 1) / TB, tiles_n3 = (a.N3 + TB - 1) / TB;
  const int per_first = tiles_m * tiles_n, per_expert = per_first + (KIND == DW_TWO ? tiles_m3 * tiles_n3 : 0);

  for (int i = threadIdx.x; i <= a.E; i += NTHREADS) s_off[i] = a.offsets ? a.offsets[i] : a.Tk / a.E * i;
  __syncthreads();
  for (int x = threadIdx.x; x < a.E; x += NTHREADS) {
    int nx = s_off[x + 1] - s_off[x], before = 0;
    for (int y = 0; y < a.E; ++y) {
      int ny = s_off[y + 1] - s_off[y];
      before += (ny > nx) || (ny == nx && y < x);
    }
    s_order[before] = x;
  }
  __syncthreads();

  // the tiles that the loader has opened, for the multiplying side; a ring per wavefront (the loader is at most two tiles ahead)
  __shared__ __attribute__((aligned(16))) int s_tile[4][4][4];
  constexpr int FURTHER = 1 << 30;
  auto rows_a = [&](const DWCursor &c) { return KIND == DW_A || KIND == DW_AB || (KIND == DW_TWO && c.further && a.a3_map.o); };
  auto rows_b = [&](const DWCursor &c) { return KIND == DW_B || KIND == DW_AB || (KIND == DW_TWO && !c.further && a.b_map.o); };
  auto open_tile = [&](DWCursor &c, int seq) {
    c.seq = seq;
    c.step = 0;
    const int U = seq * G + slot_in_round;
    const int T = split > 1 ? U / split : U;
    const int rank = T / per_expert;
    if (rank >= a.E || (split > 1 && seq > 0)) {   // past the last tile: stages without rows
      c.left = 0;
      c.ns = 0x7fffffff;
      *reinterpret_cast<int4 *>(s_tile[wave][seq & 3]) = make_int4(0, 0, 0, 0);
      return;
    }
    const int t = T - rank * per_expert;
    c.e = split > 1 ? rank : __builtin_amdgcn_readfirstlane(s_order[rank]);   // LDS reads land in vector registers: make them scalar again
    int lo = __builtin_amdgcn_readfirstlane(s_off[c.e]), hi = __builtin_amdgcn_readfirstlane(s_off[c.e + 1]);
    if (split > 1) dw_chunk_rows(lo, hi, split, U - T * split, lo, hi);
    c.further = KIND == DW_TWO && t >= per_first;
    if (c.further) dw_tile_origin(t - per_first, tiles_m3, tiles_n3, c.m0, c.n0);
    else dw_tile_origin(t, tiles_m, tiles_n, c.m0, c.n0);
    c.left = hi - lo;
    // Stages come in pairs so that every tile starts in LDS slot 0 and the loop can be written with compile-time slots; the extra
    // stage (two for an empty expert) loads zeros and adds nothing.
    c.ns = max(((c.left + SK - 1) / SK + 1) & ~1, 2);
    const bool second = KIND == DW_PAIR && c.e == 1;
    const uint32_t row_a = (uint32_t)(c.further ? a.M3 : a.M) * 2u, row_b = (uint32_t)(c.further ? a.N3 : a.N) * 2u;
    c.pa = (const char *)(c.further ? a.A3 : second ? a.A2 : a.A);
    c.pb = (const char *)(c.further ? a.B3 : second ? a.B2 : a.B);
    const bool through_a = rows_a(c), through_b = rows_b(c);
    c.sa = through_a ? 0u : SK * row_a;
    c.sb = through_b ? 0u : SK * row_b;
    if (!through_a) c.pa += (size_t)lo * row_a;
    if (!through_b) c.pb += (size_t)lo * row_b;
    if (ROWS) c.po = (KIND == DW_TWO ? a.order : KIND == DW_A ? a.a_map.o : a.b_map.o) + lo;   // every map has the same order indices
    *reinterpret_cast<int4 *>(s_tile[wave][seq & 3]) = make_int4(c.e | (c.further ? FURTHER : 0), c.m0, c.n0, c.ns);
  };
  auto follow = [&](DWTile &t, int seq) -> bool {
    const int4 v = *reinterpret_cast<const int4 *>(s_tile[wave][seq & 3]);
    const int e = __builtin_amdgcn_readfirstlane(v.x);
    t.seq = seq;
    t.e = e & ~FURTHER;
    t.further = KIND == DW_TWO && (e & FURTHER);
    t.m0 = __builtin_amdgcn_readfirstlane(v.y);
    t.n0 = __builtin_amdgcn_readfirstlane(v.z);
    t.ns = __builtin_amdgcn_readfirstlane(v.w);
    return t.ns > 0;
  };
  auto advance = [&](DWCursor &c) {
    c.left -= SK;
    c.pa += c.sa;
    c.pb += c.sb;
    if (ROWS) c.po += SK;
    if (++c.step < c.ns) return;
    // keeps the tile lookup behind this (rarely taken) branch: without it the compiler evaluates
    // the lookup's integer divisions in every stage and selects the results
    __asm__ volatile("" ::: "memory");
    open_tile(c, c.seq + 1);
  };

  DWStreamOps<KIND> ops;
  ops.uwave = __builtin_amdgcn_readfirstlane(wave);
  ops.magic_a = magic_a;
  ops.magic_b = magic_b;
  ops.row = wave * 16 + (lane >> 5);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ops.fa[q] = rows_frag_offset(wm * (TB / 2) + q * 32, lane);
    ops.fb[q] = rows_frag_offset(wn * (TB / 2) + q * 32, lane);
  }
  const uint32_t rows_lds = __builtin_amdgcn_readfirstlane(lds_address((const char *)&s_rows[0][0][0])) + (ROWS ? ops.uwave * 256 : 0);
  const uint32_t rows_lane = (uint32_t)(wave * 16 + (lane & 7) * 2 + ((lane >> 3) & 1)) * 4u;
  // rows of the segment in a stage (by hand: the compiler's median instruction is a vector one, and takes all that follows with it)
  auto stage_rows = [](const DWCursor &c) {
    uint32_t n;
    __asm__("s_max_i32 %0, %1, 0\n\ts_min_i32 %0, %0, %2" : "=&s"(n) : "s"(c.left), "n"(SK) : "scc");
    return n;
  };
  // order indices of the rows that this wavefront loads of a stage -> s_rows[parity], the even rows in front (four copies)
  auto fetch_rows = [&](const DWCursor &c, int parity) {
    load4_to_lds_checked(scalar_window(c.po, stage_rows(c) * 4u), rows_lane, rows_lds + parity * 1024);
  };
  // publishes the stage whose loads are issued next
  uint32_t row_a = 0, row_b = 0;
  auto resolve = [&](const DWCursor &c, int parity) {
    const bool through_a = rows_a(c), through_b = rows_b(c);
    if (c.step == 0) {   // a new tile
      const int M = c.further ? a.M3 : a.M, N = c.further ? a.N3 : a.N;
      row_a = (uint32_t)M * 2u;   // bytes per operand row
      row_b = (uint32_t)N * 2u;
      ops.pair_a = through_a ? 0u : 4u * row_a;
      ops.pair_b = through_b ? 0u : 4u * row_b;
      ops.mul_a = through_a ? row_a : 0u;
      ops.mul_b = through_b ? row_b : 0u;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int r = p * 2 + (lane >> 5), col = ((lane & 31) ^ tr_swz(r)) * 8;
        int ca = c.m0 + col, cb = c.n0 + col;
        if (ca >= M) ca = 0;
        if (cb >= N) cb = 0;
        ops.oa[p] = (through_a ? 0u : (uint32_t)(wave * 16 + r) * row_a) + (uint32_t)ca * 2u;
        ops.ob[p] = (through_b ? 0u : (uint32_t)(wave * 16 + r) * row_b) + (uint32_t)cb * 2u;
      }
    }
    const uint32_t rows = stage_rows(c);
    ops.win_a = scalar_window(c.pa, through_a ? MAX_SOURCE_BYTES : rows * row_a);
    ops.win_b = scalar_window(c.pb, through_b ? MAX_SOURCE_BYTES : rows * row_b);
    if (ROWS) {
      ops.left = c.left;
      const uint4 *o = reinterpret_cast<const uint4 *>(&s_rows[parity][wave][(lane >> 5) * 8]);
      const uint4 lo = o[0], hi = o[1];
      ops.order[0] = lo.x; ops.order[1] = lo.y; ops.order[2] = lo.z; ops.order[3] = lo.w;
      ops.order[4] = hi.x; ops.order[5] = hi.y; ops.order[6] = hi.z; ops.order[7] = hi.w;
    }
  };

  DWCursor lc;
  DWTile cc;
  open_tile(lc, 0);
  if (!follow(cc, 0)) return;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
  char *patch = smem + Big::RING_BYTES + ops.uwave * EPI_WAVE_BYTES;
  DWCursor rc = lc;                           // ROWS: the stage whose order indices are fetched next
  auto fetch_next = [&](int parity) {
    if (!ROWS) return;
    fetch_rows(rc, parity);
    advance(rc);
  };
  fetch_next(0);
  fetch_next(1);
  if (ROWS) wait_loads<0>();
#pragma unroll 1
  for (int st = 0; st < Big::SLOTS; ++st) {
    resolve(lc, st);
#pragma unroll
    for (int I = 0; I < Big::NL; ++I) ops.load(I, lds0 + st * Big::A_BYTES, lds0 + Big::SLOTS * Big::A_BYTES + st * B_BYTES);
    advance(lc);
    if (st == 0) fetch_next(0);               // in front of the second stage's loads, like all later ones
  }
  wait_loads<(Big::SLOTS - 1) * Big::NL>();   // the first stage has landed
  __syncthreads();
  resolve(lc, 0);
  if (ROWS) {
    advance(lc);
    fetch_rows(lc, 1);
  }
  f32x16 acc[FR][FR];
  Frags<Big> f[4];
#pragma unroll
  for (int i = 0; i < Big::NF; ++i) read_item<Big>(ops, f[0], i, smem, smem + Big::SLOTS * Big::A_BYTES, 0);

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // Behind the stage in slot `cur`: the operands of the loads that the next stage issues.  With ROWS the cursor is one stage further,
  // that of the indices fetched here; the ones read here landed at the wait of the stage just done.
  auto next_stage = [&](int cur) {
    if (ROWS) {
      resolve(lc, cur ^ 1);
      advance(lc);
      fetch_rows(lc, cur);
    } else {
      advance(lc);
      resolve(lc, 0);
    }
  };
  for (;;) {   // one tile per trip
    // the stores of the previous tile's epilogue lie behind the loads that the first stage's wait is for
    if (cc.seq > 0) stage_step<true, false, EpilogueStores<Big::FM, 0>, Big>(ops, f, acc, smem, lds0, I0{}, I1{});
    else stage_step<true, false, 0, Big>(ops, f, acc, smem, lds0, I0{}, I1{});
    next_stage(0);
    stage_step<false, false, 0, Big>(ops, f, acc, smem, lds0, I1{}, I0{});
    next_stage(1);
    for (int h = 2; h < cc.ns; h += 2) {
      stage_step<false, false, 0, Big>(ops, f, acc, smem, lds0, I0{}, I1{});
      next_stage(0);
      stage_step<false, false, 0, Big>(ops, f, acc, smem, lds0, I1{}, I0{});
      next_stage(1);
    }
    const int mbase = cc.m0 + uwm * (TB / 2), wcol = cc.n0 + uwn * (TB / 2);
    if (split > 1) {
      store_wave_partial(acc, a.split_ws + (size_t)(cc.seq * G + slot_in_round) * TB * TB + (size_t)(uwm * (TB / 2)) * TB + uwn * (TB / 2), lane);
    } else {
      const int M = KIND == DW_TWO && cc.further ? a.M3 : a.M, N = KIND == DW_TWO && cc.further ? a.N3 : a.N;
      const uint32_t row_b = (uint32_t)N * 2u;
      const int left = max(min(TB / 2, M - mbase), 0);
      const window_t win = make_window((const bf16_t *)(KIND == DW_TWO && cc.further ? a.dW3 : DENSE_PAIR && cc.e == 1 ? a.dW2 : a.dW) + (size_t)cc.e * M * N + (size_t)min(mbase, M) * N, (uint32_t)left * row_b);
      store_wave_tile(acc, patch, [&](int fm, int half) {
        BlockDest d{win, {}};
        const int col = wcol + half * 64 + (lane & 7) * 8;
        const uint32_t mine = col < N ? (uint32_t)(lane >> 3) * row_b + (uint32_t)col * 2u : OFF_WINDOW;
#pragma unroll
        for (int it = 0; it < 4; ++it) d.off[it] = mine + (uint32_t)(fm * 32 + it * 8) * row_b;
        return d;
      }, lane);
    }
    if (!follow(cc, cc.seq + 1)) break;
  }
  wait_loads<0>();
}

// Second pass of a row-split groupXTY: adds each tile's partials in chunk order, rounds once, stores dW.
__global__ void __launch_bounds__(256) dw_split_reduce_kernel(DWArgs a, int tiles_m, int tiles_n, int split) {
  const int per_expert = tiles_m * tiles_n;
  const int T = blockIdx.x, e = T / per_expert;
  int m0, n0;
  dw_tile_origin(T - e * per_expert, tiles_m, tiles_n, m0, n0);
  const float *part = a.split_ws + (size_t)T * split * TB * TB;
  bf16_t *dW = (bf16_t *)(a.dW2 && e == 1 ? a.dW2 : a.dW) + (size_t)e * a.M * a.N;
  constexpr int PER_SLICE = TB * TB / 4 / TAIL_SLICES;
  for (int i = (int)blockIdx.y * PER_SLICE + threadIdx.x; i < ((int)blockIdx.y + 1) * PER_SLICE; i += 256) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int c = 0; c < split; ++c) {
      const float4 v = reinterpret_cast<const float4 *>(part + (size_t)c * TB * TB)[i];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    const int row = m0 + (i * 4) / TB, col = n0 + (i * 4) % TB;
    if (row < a.M && col < a.N) {
      bf16x4 o;
      o[0] = (bf16_t)acc.x; o[1] = (bf16_t)acc.y; o[2] = (bf16_t)acc.z; o[3] = (bf16_t)acc.w;
      *reinterpret_cast<bf16x4 *>(dW + (size_t)row * a.N + col) = o;
    }
  }
}

template <typename S, bool TRANS_W, bool SCATTER_OUT, int ACT, bool STATIC2, bool WIDE> int launch_s2s_one(hipStream_t s, const S2SArgs &a) {
  const int tiles_n = (ACT == 1 || ACT == 2) ? ceil_div(a.N / 2, TB / 2) : ceil_div(a.N, TB);
  const long long tiles_m = ceil_div(a.Tk, S::TM) + a.E;     // upper bound on sum_e ceil(n_e / TM)
  const int group_m = a.group_m * (TB / S::TM), grid = a.grid;
  if (tiles_m * tiles_n > 0x7fffffffLL) return SMOE_ERR_UNSUPPORTED;
  S2SArgs args = a;
  int chunk;
  if (ACT != 0 || choose_split(ceil_div(a.K, SK), 4, STATIC2, chunk) == 1) args.tail_ws = nullptr;   // too short to pay: no second kernel
  hipLaunchKernelGGL((s2s_stream_kernel<S, TRANS_W, SCATTER_OUT, ACT, STATIC2, WIDE>), dim3(grid), dim3(NTHREADS), S::LDS_BYTES, s, args,
                     tiles_n, group_m, division_magic(a.a_map.o ? a.a_map.fan : 1));
  SMOE_LAUNCH_CHECK();
  if (args.tail_ws) {   // adds and stores the partial tiles of a split last round (no-op when nothing was split)
    hipLaunchKernelGGL((s2s_tail_reduce_kernel<S, SCATTER_OUT>), dim3(TAIL_BLOCKS), dim3(256), 0, s, a, tiles_n, group_m, grid, STATIC2 ? 1 : 0);
    SMOE_LAUNCH_CHECK();
  }
  return SMOE_OK;
}
// Which shape a launch takes.  The row counts are on the device, so an expert is taken to have r = Tk / E rows: r / TM + 1/2
// tiles on average, one when it has few rows.  Estimated time in microseconds: a stage 1.5 (Big), 0.9 (Half), epilogue and tile set-up
// 6 / 4; a split's partial tiles written and read at 4.5 TB/s, and 5 for the second kernel.  Half is taken where that promises 5 %
// (at 1 % it lost as often as it won).  Measured, Big / Half in us:
//   8192 rows, 8 experts: 1024 -> 2 x 2816 with SwiGLU 132 / 114 where a row more makes a fourth round of the big tiles, 100 / 114
//   where not; its W1^T counterpart (5632 -> 1024) 134 / 106; 2816 -> 1024 72 / 75;  6002 rows, 3416 -> 1280: 95 / 59;
//   6832 -> 1280 W^T 188 / 123;  2 x 8192 rows: 2048 -> 512 54 / 34;  32768 rows, 16 experts: 2048 -> 512 92 / 88, 512 -> 2048 84 / 91;
//   65536 rows, 64 experts: 2048 -> 2 x 512 with SwiGLU 268 / 308, 512 -> 2048 152 / 183, 1024 -> 2048 W^T 287 / 325;
//   262144 rows, 64 experts: 4096 -> 512 930 / 1060;  32768 rows, 8 experts: 14336 -> 4096 3020 / 3530;
//   32768 rows, 16 experts, 2048 -> 512 W^T with dp and the weighted rows in the epilogue (ACT 6) 121 / 105.
// Even loads make the next whole number of tiles instead, which a long contraction that stands at the end of a round pays dearly for:
// contractions over 2048 take Half only where the mean over both counts says so too.  2937 tokens on 37 experts, k = 6, 7808 -> 720: 262 big
// tiles by the first count, a round and a bit, 222 by the second; Big 232, Half 283.  Whole forward passes with / without that: this
// one 589 / 641, 3150 tokens on 31 experts, k = 4, 2496 -> 6336, 1298 / 1369, 794 on 48, k = 8, 3840 -> 2 x 1216, 335 / 352, the worst (1046 on 11,
// k = 8, 2112 -> 2944, forward and backward) 1139 / 1127.  Under 2048 the mean lost as often as it won.
template <typename S> long long estimated_tiles(const S2SArgs &a, int tiles_n, bool even = false) {
  const float rows = (float)a.Tk / a.E;
  const float m_tiles = even || a.E == 1 || a.C2 ? (float)ceil_div(ceil_div(a.Tk, a.E), S::TM) : rows >= S::TM ? rows / S::TM + 0.5f : 1.0f;
  return (long long)(m_tiles * (a.Tk < a.E ? a.Tk : a.E) * tiles_n + 0.5f);
}
template <typename S> float launch_estimate(const S2SArgs &a, int tiles_n, bool static2, bool may_split, bool even) {
  const int ns = ceil_div(a.K, SK), G = a.grid;
  const long long total = estimated_tiles<S>(a, tiles_n, even);
  const float full = S::FM > 2 ? 1.5f * ns + 6.f : 0.9f * ns + 4.f;
  const int rest = (int)(total % G);
  float t = (total / G) * full;
  int chunk = ns, split = 1;
  if (rest > 0) {
    if (may_split) split = choose_split(ns, G / rest, static2, chunk);
    t += full / split;
  }
  if (split > 1) t += 5.f + rest * split * (S::PART * 8.f / 4.5e6f);
  return t;
}
bool prefer_half(const S2SArgs &a, int tiles_n, bool may_split) {
  const bool static2 = a.K % (2 * SK) == 0;
  const float half = launch_estimate<Half>(a, tiles_n, false, may_split, false), big = launch_estimate<Big>(a, tiles_n, static2, may_split, false);
  if (half >= 0.95f * big || a.K <= 2048) return half < 0.95f * big;
  return half + launch_estimate<Half>(a, tiles_n, false, may_split, true) < 0.95f * (big + launch_estimate<Big>(a, tiles_n, static2, may_split, true));
}
template <bool TRANS_W, bool SCATTER_OUT, int ACT = 0> int launch_s2s_cfg(hipStream_t s, const S2SArgs &a) {
  const bool static2 = a.K % (2 * SK) == 0;
  if constexpr (SCATTER_OUT && ACT == 0)
    if ((long long)a.Tk * a.N * 2 > 0xfffffff0LL) {   // rows a 32-bit offset does not reach
      if (static2) return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, true, true>(s, a);
      return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, false, true>(s, a);
    }
  const int tiles_n = (ACT == 1 || ACT == 2) ? ceil_div(a.N / 2, TB / 2) : ceil_div(a.N, TB);
  const bool may_split = ACT == 0 && a.tail_ws;
  if (a.tile_shape == 1 || (a.tile_shape == 0 && prefer_half(a, tiles_n, may_split))) {
    // At most one tile row per expert on average: most of W is read once, and where the call's weights exceed the last-level cache
    // keeping its lines only pushes other data out; a tile of an expert that has several reads what the others do and takes it the
    // ordinary way (777 tokens on 64 experts, 2048 -> 2 x 512 -> 2048, other weights at every call, the forward pass: 106 us with W
    // through the caches, 94 so; with Zipf(1.2) loads 129, 131 with all of W past them, 121 so).
    if constexpr (!TRANS_W) {
      const bool once = (long long)a.Tk <= (long long)a.E * Half::TM && weights_pass_caches(a);
      // HalfShort: contractions of up to four stages, and launches of one round whose contraction is up to eight or which read most of W
      // once by rows at a stride of whole kilobytes.  Few stages are over before a third slot's requests come in; and a block with a
      // single tile waits for W at every stage, where requests for many rows that fall on few cache sets wait for one another (the
      // more so with SwiGLU, which reads each row in two places).  Two / three slots in us, W from memory (from the last-level cache), 16
      // experts of 62 rows, SwiGLU: 512 -> 2 x 512 15.2 / 15.7, 2048 -> 2 x 512 39.6 / 40.8 (33.6 / 35.5), 4096 -> 2 x 512 69.5 / 71.6 (59.5 / 63.3);
      // 37 experts of 60 rows, 3840 -> 512 61.9 / 63.6, 64 of 97 rows, 2048 -> 1024 54.5 / 55.6; 16 experts of 256 rows, 128 -> 2048 11.7 / 12.7.
      // Elsewhere the third slot is worth more: other strides, 16 of 62 rows, 2048 -> 2 x 448 37.1 / 34.5; W read several times, 4 of 292 rows,
      // 2688 -> 2048 43.7 / 41.2; several rounds, 16 of 1024 rows, 4096 -> 2 x 2816 796 / 750.
      const bool one_round = estimated_tiles<Half>(a, tiles_n) <= a.grid, apart = a.ldw % 512 == 0 && (long long)a.Tk <= (long long)a.E * Half::TM;
      if (a.K <= 4 * SK || (one_round && (a.K <= 8 * SK || apart))) {
        if (once) return launch_s2s_one<HalfShortOnce, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
        return launch_s2s_one<HalfShort, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
      }
      if (once) return launch_s2s_one<HalfOnce, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
    }
    return launch_s2s_one<Half, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
  }
  if (static2) return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, true, false>(s, a);
  return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
}

int launch_dw_stream_impl(hipStream_t s, const DWArgs &a) {
  int tiles_m = ceil_div(a.M, TB), tiles_n = ceil_div(a.N, TB);
  // Row split: only when every tile of every expert, times the split, fits one round of the grid, and only when
  // it shortens the contraction by more than the partial tiles cost (as for the split last round above).
  int split = 1;
  const long long tiles = (long long)a.E * tiles_m * tiles_n;
  if (a.split_ws && tiles * 2 <= a.grid) {
    const long long ns = a.Tk / a.E / SK;            // stages of an average segment
    split = (int)(a.grid / tiles < 8 ? a.grid / tiles : 8);
    if (ns - ns / split < SPLIT_MIN_SAVED) split = 1;
  }
  if (a.dW3) split = 1;
  auto magic = [](int fan) { return (uint32_t)((0x80000000ULL + fan - 1) / fan); };   // of twice the dividend: exact while Tk * fan < 2^31
  const uint32_t magic_a = magic(a.dW3 ? a.a3_map.fan : a.a_map.fan), magic_b = magic(a.b_map.fan);
  auto launch = [&](auto kind) {
    hipLaunchKernelGGL(dw_stream_kernel<decltype(kind)::value>, dim3(a.grid), dim3(NTHREADS), Big::LDS_BYTES, s, a, tiles_m, tiles_n, split, magic_a, magic_b);
  };
  if (a.dW3) launch(std::integral_constant<int, DW_TWO>{});
  else if (a.dW2) launch(std::integral_constant<int, DW_PAIR>{});
  else if (a.a_map.o && a.b_map.o) launch(std::integral_constant<int, DW_AB>{});
  else if (a.a_map.o) launch(std::integral_constant<int, DW_A>{});
  else if (a.b_map.o) launch(std::integral_constant<int, DW_B>{});
  else launch(std::integral_constant<int, DW_ONE>{});
  SMOE_LAUNCH_CHECK();
  if (split > 1) {
    hipLaunchKernelGGL(dw_split_reduce_kernel, dim3((unsigned)tiles, TAIL_SLICES), dim3(256), 0, s, a, tiles_m, tiles_n, split);
    SMOE_LAUNCH_CHECK();
  }
  return SMOE_OK;
}
}  // namespace

// A tile must have at least two stages (the index ring assumes it); the expert offsets must fit their LDS cache; order
// indices are divided by the fan-out with a multiply-high that is exact while Tk * fan < 2^32.  Every source offset (from
// the start of a gathered A, of an expert's matrix, of a tile's first row) must fit 32 bits with the last stage's
// overhang, and a tile's rows of an output 31 bits.
bool s2s_stream_supported(const S2SArgs &a) {
  const long long fan = a.a_map.o ? a.a_map.fan : 1;
  const long long a_rows = a.a_map.o ? (long long)a.Tk / fan + 1 : TB;
  const long long w_rows = a.trans_w ? a.N : a.K;
  return a.grid >= 8 && a.grid % 8 == 0 && a.grid <= MAX_STREAM_GRID && a.group_m >= 1 && a.K % 8 == 0 && a.K > SK && a.N % 8 == 0 &&
         a.ldw % 8 == 0 && a.Tk > 0 && a.E <= MAX_E && (long long)a.Tk * fan < 0x100000000LL && (a_rows * a.K + SK) * 2 < 0x100000000LL &&
         (w_rows + SK) * a.ldw * 2 < 0x100000000LL && (long long)TB * a.N * 4 < 0x80000000LL;
}
bool s2s_stream_swiglu_bwd_supported(const S2SArgs &a) {
  return s2s_stream_supported(a) && a.trans_w && a.a_map.o && !a.c_map.o && a.Hpre_in && (!a.Hw_out || a.H_in) && a.row_scale && a.dp_part && a.N % 8 == 0;
}

bool s2s_stream_dp_supported(const S2SArgs &a) {
  const bool slots_fit = !a.c_map.o || (a.Hw_out && (long long)a.Tk * a.N * 2 <= 0xfffffff0LL);   // ACT 6: 32-bit offsets of slot rows
  return s2s_stream_supported(a) && a.trans_w && a.a_map.o && slots_fit && a.H_in && !a.Hpre_in && a.row_scale && a.dp_part && a.N % 8 == 0;
}

bool s2s_stream_swiglu_supported(const S2SArgs &a) {
  return s2s_stream_supported(a) && !a.trans_w && !a.c_map.o && a.H && a.N % 16 == 0;
}

int launch_s2s_stream(hipStream_t s, const S2SArgs &a) {
  const bool scatter_out = a.c_map.o != nullptr;
  if (a.dp_part && a.Hpre_in) {
    if (!s2s_stream_swiglu_bwd_supported(a)) return SMOE_ERR_UNSUPPORTED;
    return a.Hw_out ? launch_s2s_cfg<true, false, 7>(s, a) : launch_s2s_cfg<true, false, 3>(s, a);
  }
  if (a.dp_part) {
    if (!s2s_stream_dp_supported(a)) return SMOE_ERR_UNSUPPORTED;
    if (scatter_out) return launch_s2s_cfg<true, true, 6>(s, a);
    return a.Hw_out ? launch_s2s_cfg<true, false, 5>(s, a) : launch_s2s_cfg<true, false, 4>(s, a);
  }
  if (a.H) {
    if (!s2s_stream_swiglu_supported(a)) return SMOE_ERR_UNSUPPORTED;
    return a.C ? launch_s2s_cfg<false, false, 1>(s, a) : launch_s2s_cfg<false, false, 2>(s, a);
  }
  if (a.trans_w) return scatter_out ? launch_s2s_cfg<true, true>(s, a) : launch_s2s_cfg<true, false>(s, a);
  return scatter_out ? launch_s2s_cfg<false, true>(s, a) : launch_s2s_cfg<false, false>(s, a);
}

// Rows that groupXTY reads through the order indices: 32-bit offsets from the source's start, made by a 24-bit multiplication, and a
// division by the fan-out that is exact while Tk * fan < 2^31.
static bool rows_readable(const RowMap &m, int Tk, int width) {
  if (!m.o) return true;
  const long long rows = Tk / m.fan, bytes = (long long)width * 2;
  return rows < (1 << 24) && bytes < (1 << 24) && rows * bytes <= (long long)MAX_SOURCE_BYTES && (long long)Tk * m.fan < 0x80000000LL;
}
bool dw_stream_supported(const DWArgs &a) {
  long long tiles = (long long)a.E * ((long long)ceil_div(a.M, TB) * ceil_div(a.N, TB) + (long long)ceil_div(a.M3, TB) * ceil_div(a.N3, TB));
  return a.M % 8 == 0 && a.N % 8 == 0 && a.M3 % 8 == 0 && a.N3 % 8 == 0 && a.Tk > 0 && a.E <= MAX_E && tiles + MAX_STREAM_GRID < 0x7fffffffLL && a.grid >= 8 &&
         a.grid % 8 == 0 && a.grid <= MAX_STREAM_GRID && (long long)TB * a.N * 2 < 0x80000000LL && (long long)TB * a.N3 * 2 < 0x80000000LL &&
         rows_readable(a.a_map, a.Tk, a.M) && rows_readable(a.b_map, a.Tk, a.N) && rows_readable(a.a3_map, a.Tk, a.M3) &&
         !(a.dW2 && (a.a_map.o || a.b_map.o)) &&
         // beside dW3 the order indices are fetched for every stage, from `order`, also where both operands lie sorted
         (!a.dW3 || (a.order && !a.a_map.o && (!a.b_map.o || a.b_map.o == a.order) && (!a.a3_map.o || a.a3_map.o == a.order)));
}

// Together two weight gradients save the rounds that their last tiles fill only in part, and a launch, while a stage costs 3 % more
// (its operands are chosen).  8 experts of 750 rows, 3416 x 1280 and 1280 x 6832 (2.2 + 4.2 rounds of tiles): 81 + 145 -> 203 us.  Whole
// backward passes in us, one launch for each / one for both, where a round is saved: those 8 experts 584 / 559, with Zipf(1.2) loads 614 /
// 575, with 20000 rows 1390 / 1352; 24000 rows and Zipf loads 1705 / 1566; 4 experts, 1280 -> 2 x 2048, 6000 rows 303 / 257; 16 experts,
// 1280 -> 2 x 1024, 12000 rows 295 / 270; 64 experts, 768 -> 512, 8000 rows 130 / 111; 16 experts, 1280 -> 2 x 3416 (14 rounds to 13),
// 24000 rows 1632 / 1612.
bool dw_stream_two_pay(const DWArgs &a) {
  const long long first = (long long)a.E * ceil_div(a.M, TB) * ceil_div(a.N, TB), further = (long long)a.E * ceil_div(a.M3, TB) * ceil_div(a.N3, TB);
  auto rounds = [&](long long tiles) { return (tiles + a.grid - 1) / a.grid; };
  if (first * 2 <= a.grid || further * 2 <= a.grid) return false;      // one of them may be cut along its rows instead
  return rounds(first + further) * 33 <= (rounds(first) + rounds(further)) * 32;
}

int launch_dw_stream(hipStream_t s, const DWArgs &a) { return launch_dw_stream_impl(s, a); }

// Raises the dynamic LDS limit of every persistent kernel on the current device (once per context).
template <bool TRANS_W, bool SCATTER_OUT, int ACT> static int init_s2s() {
  int rc = set_lds_limit(s2s_stream_kernel<Big, TRANS_W, SCATTER_OUT, ACT, true, false>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<Big, TRANS_W, SCATTER_OUT, ACT, false, false>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<Half, TRANS_W, SCATTER_OUT, ACT, false, false>, Half::LDS_BYTES);
  if constexpr (!TRANS_W) {
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<HalfOnce, TRANS_W, SCATTER_OUT, ACT, false, false>, HalfOnce::LDS_BYTES);
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<HalfShort, TRANS_W, SCATTER_OUT, ACT, false, false>, HalfShort::LDS_BYTES);
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<HalfShortOnce, TRANS_W, SCATTER_OUT, ACT, false, false>, HalfShortOnce::LDS_BYTES);
  }
  if constexpr (SCATTER_OUT && ACT == 0) {
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<Big, TRANS_W, SCATTER_OUT, ACT, true, true>, Big::LDS_BYTES);
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<Big, TRANS_W, SCATTER_OUT, ACT, false, true>, Big::LDS_BYTES);
  }
  return rc;
}
int init_stream_kernels() {
  int rc = init_s2s<false, false, 0>();
  if (rc == SMOE_OK) rc = init_s2s<false, true, 0>();
  if (rc == SMOE_OK) rc = init_s2s<true, false, 0>();
  if (rc == SMOE_OK) rc = init_s2s<true, true, 0>();
  if (rc == SMOE_OK) rc = init_s2s<false, false, 1>();
  if (rc == SMOE_OK) rc = init_s2s<false, false, 2>();
  if (rc == SMOE_OK) rc = init_s2s<true, false, 3>();
  if (rc == SMOE_OK) rc = init_s2s<true, false, 4>();
  if (rc == SMOE_OK) rc = init_s2s<true, false, 5>();
  if (rc == SMOE_OK) rc = init_s2s<true, true, 6>();
  if (rc == SMOE_OK) rc = init_s2s<true, false, 7>();
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_ONE>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_A>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_B>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_AB>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_PAIR>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_TWO>, Big::LDS_BYTES);
  return rc;
}
