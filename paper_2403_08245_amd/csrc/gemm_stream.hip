// Persistent ("stream") form of the bf16 matrix-core grouped GEMMs.
//
// Blocks walk lists of output tiles.  The LDS ring of the contraction loop never drains between tiles: the loader runs
// several half-steps (of 32 contraction elements) ahead of the multiplying side and simply moves on to the next tile's
// operand rows, so the next tile's first stages land while the current tile is being finished and written out.
//
// A half-step has two phases.  Phase A issues the first half's matrix instructions from fragments that are already in
// registers and reads the second half's fragments behind them; then, in the MIDDLE of the half-step, comes the only
// barrier: every wavefront holds all of the stage's fragments, so its slot is free, and the next stage has landed.  Phase
// B multiplies the second half, reads the next stage's first fragments, and starts to refill the freed slot; the refill
// ends in the next phase A.  With the barrier in the middle a ring of S slots keeps almost S half-steps of loads in flight
// (at the start of a half-step it would be S - 2 and a bit: the slot just left could only be refilled a half-step later).
//
// Two shapes (Shape below):
//   Big   256 x 256 tiles, four 32 KB slots, one block per compute unit (one wavefront per SIMD, 256 accumulators): the
//         fewest operand bytes per multiply-add.
//   Pair  128 x 256 tiles, three 24 KB slots, two blocks per compute unit (128 accumulators, at most 256 registers): one
//         block's epilogue, barriers and fragment reads run under the other's matrix instructions, and half as many rows
//         per tile waste fewer rows at segment ends and leave less work over when the tiles do not fill a last round; the
//         price is 1.5 times the operand traffic.
//
// Loads are inline assembly so that the waits are placed by hand; stores share the hardware counter with them and complete
// in order, and because every epilogue issues a known number of stores at least, the first waits after an epilogue step
// over them instead of sitting out their acknowledgement.  All loads go through range-checked buffer windows: rows past a
// segment and contraction elements past K read zeros.  Row indices travel through LDS by direct-to-LDS loads as well: no
// ordinary global load sits in the loop, so the compiler never inserts a full wait in front of the loads in flight.
#include "gemm_epilogue.h"
#include <type_traits>

namespace {

template <int FM_, int SLOTS_, int BLOCKS_, bool ONCE_ = false> struct Shape {
  static constexpr int FM = FM_;                        // 32-row fragments per wavefront (2 x 2 wavefronts, FR = 4 column fragments)
  static constexpr int TM = FM * 64;                    // tile rows; tile columns are TB = 256
  static constexpr int A_BYTES = TM * HK * 2;
  static constexpr int SLOT_BYTES = A_BYTES + TILE_BYTES;
  static constexpr int SLOTS = SLOTS_;
  static constexpr int BLOCKS = BLOCKS_;                // blocks per compute unit
  static constexpr bool ONCE = ONCE_;                   // W is read past the caches
  static constexpr int NLA = FM;                        // load instructions per wavefront and stage: A part,
  static constexpr int NL = NLA + NLD;                  // both parts
  static constexpr int HALF = NL / 2;                   // issued in phase B; the rest in the next phase A
  static constexpr int IN_FLIGHT = (SLOTS - 2) * NL;    // loads issued after those of the next stage, in the middle of a half-step
  static constexpr int PART = TM * TB;                  // elements of an fp32 partial tile
  // With two blocks per compute unit the patch of an epilogue is the part of the finished slot that the wavefront loads
  // itself: nobody else touches it until the same wavefront issues that slot's next loads, held back until after the
  // epilogue.  The big tile has LDS for a patch of its own and lets its loads run on.
  static constexpr bool PATCH_IN_SLOT = BLOCKS > 1;
  static constexpr int LDS_BYTES = SLOTS * SLOT_BYTES + (PATCH_IN_SLOT ? 0 : 4 * EPI_WAVE_BYTES);
};
using Big = Shape<4, 4, 1>;
using Pair = Shape<2, 3, 2>;
using PairOnce = Shape<2, 3, 2, true>;
constexpr int MAX_STREAM_GRID = 256;                    // compute units used; the partial-tile scratch holds this many big tiles

template <typename S> struct Frags {                    // one wavefront's fragments for 16 contraction elements
  bf16x8 a[S::FM], b[FR];
};
template <typename S, typename Ops>
__device__ __forceinline__ void read_frag_group(const Ops &ops, Frags<S> &f, const char *slot, int kk, int group, int wm, int wn, int lane) {
  auto A = [&](int i) { f.a[i] = ops.frag_a(slot, wm * (S::TM / 2) + i * 32, kk, lane); };
  auto B = [&](int j) { f.b[j] = ops.frag_b(slot + S::A_BYTES, wn * (TB / 2) + j * 32, kk, lane); };
  // in the order the next phase consumes them: b0 a0 b1 | b2 b3 a1 | a2 a3
  if (group == 0) { B(0); A(0); B(1); }
  if (group == 1) { B(2); B(3); A(1); }
  if (group == 2 && S::FM == 4) { A(2); A(3); }
}
// Phase A (KK = 0) or B (KK = 1): multiplies `use`, reads `next` from `slot` behind the products (READ), and issues its half
// of a stage's loads into `fill`, spread over the products (LOAD).  FIRST: the tile's first products overwrite the accumulators.
template <int KK, bool FIRST, bool READ, bool LOAD, typename S, typename Ops>
__device__ __forceinline__ void phase(const Ops &ops, const Frags<S> &use, Frags<S> &next, const char *slot, uint32_t fill, int wm, int wn,
                                      int lane, f32x16 (&acc)[S::FM][FR]) {
  f32x16 zero;
#pragma unroll
  for (int q = 0; q < 16; ++q) zero[q] = 0.f;
  constexpr int LO = KK == 1 ? 0 : S::HALF, N = KK == 1 ? S::HALF : S::NL - S::HALF;
  sched_fence();
#pragma unroll
  for (int m = 0; m < S::FM; ++m) {
#pragma unroll
    for (int n = 0; n < FR; ++n)
      acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(use.b[n], use.a[m], FIRST ? zero : acc[m][n], 0, 0, 0);
    if (READ) read_frag_group<S>(ops, next, slot, 1 - KK, m, wm, wn, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    sched_fence();
    if (LOAD) {
#pragma unroll
      for (int I = LO + (m * N + S::FM - 1) / S::FM; I < LO + ((m + 1) * N + S::FM - 1) / S::FM; ++I) ops.load(I, fill);
      sched_fence();
    }
  }
}

// The contraction side shared by the kernels below: ring position, fragments, waits.
template <typename S> struct Ring {
  static constexpr uint32_t END = (S::SLOTS - 1) * S::SLOT_BYTES;
  __device__ static uint32_t after(uint32_t slot) { return slot == END ? 0u : slot + S::SLOT_BYTES; }
  __device__ static uint32_t before(uint32_t slot) { return slot == 0u ? END : slot - S::SLOT_BYTES; }
};
// In the middle of a half-step: the next stage has landed for every wavefront, and all of this stage's fragments are in
// registers.  STORES: that many stores were issued after the next stage's loads at least.
template <typename S, int STORES> __device__ __forceinline__ void middle() {
  constexpr int N = S::IN_FLIGHT + STORES;
  wait_loads<(N < 63 ? N : 63)>();
  __syncthreads();
}

// ======================================================================================
// scatter2scatter
// ======================================================================================
// How the tiles of a launch are dealt to the G blocks.  Tiles are numbered densely (tile_coords); full rounds deal G tiles.
// Of the rem < G tiles left, with two blocks per compute unit the first G / 2 go one to a compute unit (`whole`), and what
// remains beyond them (or all of rem) would keep few compute units busy for a whole tile: its contraction is cut into
// `split` chunks of `chunk` half-steps for the blocks still free; the chunks leave fp32 partial tiles that a second kernel
// adds in chunk order (deterministic) and stores.
struct TilePlan {
  int m_tiles, rounds, whole, rest, split, chunk;
};
template <typename S>
__device__ __forceinline__ TilePlan plan_tiles(const int32_t *offsets, int E, int tiles_n, int nh, int G, bool static4, bool may_split,
                                               int lane) {
  int sum = 0;
  for (int c0 = 0; c0 < E; c0 += 64) {
    int x = c0 + lane;
    int n = x < E ? (offsets[x + 1] - offsets[x] + S::TM - 1) / S::TM : 0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) n += __shfl_xor(n, d, 64);
    sum += n;
  }
  TilePlan p;
  p.m_tiles = __builtin_amdgcn_readfirstlane(sum);
  const long long total = (long long)p.m_tiles * tiles_n;
  p.rounds = (int)(total / G);
  const int rem = (int)(total - (long long)p.rounds * G), half = G / S::BLOCKS;
  p.whole = S::BLOCKS > 1 && rem > half ? half : 0;
  p.rest = rem - p.whole;
  p.split = 1;
  p.chunk = nh;
  if (may_split && p.rest > 0) p.split = choose_split(nh, (p.whole ? G - half : G) / p.rest, static4, p.chunk);
  return p;
}

// Sources of the loader's current tile: range-checked windows, and per-lane 32-bit byte offsets at contraction offset 0.
template <typename S, bool TRANS_W, bool KTAIL> struct S2SOps {
  int32x4 win_a, win_b;
  uint32_t oa[S::NLA], ob[NLD];
  uint32_t ta[S::NLA], tb[NLD];      // KTAIL: all ones where the lane's chunk of the last half-step lies past K
  uint32_t b_step;                   // bytes the W source moves per half-step
  int step, last;                    // half-step the next loads fetch; the contraction's last half-step
  int uwave;
  int again;                         // S::ONCE: above 0 where the expert has further tiles, which read the same weights
  __device__ __forceinline__ void load(int I, uint32_t slot_lds) const {
    if (I < S::NLA) {
      uint32_t off = oa[I] + (uint32_t)step * (HK * 2);
      if (KTAIL) off |= step == last ? ta[I] : 0u;
      load16_to_lds_checked(win_a, off, slot_lds + (uwave * S::NLA + I) * 1024);
    } else {
      const int J = I - S::NLA;
      uint32_t off = ob[J] + (uint32_t)step * b_step;
      if (KTAIL && TRANS_W) off |= step == last ? tb[J] : 0u;
      const uint32_t lds = slot_lds + S::A_BYTES + (uwave * NLD + J) * 1024;
      if (S::ONCE) load16_to_lds_checked_or_once(win_b, off, lds, again);
      else load16_to_lds_checked(win_b, off, lds);
    }
  }
  __device__ __forceinline__ bf16x8 frag_a(const char *tile, int base, int kk, int lane) const { return kc_frag(tile, base, kk, lane); }
  __device__ __forceinline__ bf16x8 frag_b(const char *tile, int base, int kk, int lane) const {
    return TRANS_W ? kc_frag(tile, base, kk, lane) : tr_frag(tile, base, kk, lane);
  }
};

// ACT 1: fused SwiGLU keeping the pre-activation, 2: without, 3: fused SwiGLU derivative and dp (the W2^T input-gradient
// product of Alg. 3's backward, see store_wave_tile_swiglu_bwd), 4: dp from the saved H in that product's epilogue for any
// activation (store_wave_tile_dp), 5: 4 with the routing-weighted hidden rows written as well, 6: 5 with H and dH in slot order.
// STATIC4 (Big only): the contraction is a multiple of four half-steps, so every tile starts in LDS slot 0 and the loop is
// written out four half-steps at a time with the slot as a compile-time constant: all LDS addresses become a loop-invariant
// register plus an immediate.  Without it the contraction may be any multiple of 8 (KTAIL masks the last half-step).
// WIDE: a scattered output of 4 GB or more.
template <typename S, bool TRANS_W, bool SCATTER_OUT, int ACT, bool STATIC4, bool WIDE>
__global__ void __launch_bounds__(NTHREADS, S::BLOCKS) s2s_stream_kernel(S2SArgs a, int tiles_n, int group_m, uint32_t magic_a) {
  constexpr bool SWIGLU = ACT == 1 || ACT == 2;
  constexpr bool KTAIL = !STATIC4;
  constexpr bool DENSE_PAIR = ACT == 0 && !SCATTER_OUT;   // S2SArgs::C2 may be set
  constexpr int STORES = EpilogueStores<S::FM, ACT>;
  static_assert(!SWIGLU || (!TRANS_W && !SCATTER_OUT), "the fused activation belongs to the forward, sorted-output product");
  static_assert(ACT < 3 || (TRANS_W && SCATTER_OUT == (ACT == 6)), "the fused derivative belongs to the W^T product");
  static_assert(!STATIC4 || S::SLOTS == 4, "the unrolled loop walks four slots");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int s_off[MAX_E + 1];
  // Order indices of the rows of up to four open tiles.  With the shortest contraction the kernel takes (three
  // half-steps) the loader has opened tile n+2 and requested the rows of tile n+3 while tile n's epilogue still
  // reads its destination rows, so four entries are live at once.
  __shared__ int s_idx[4][S::TM];
  // The open tiles themselves, left by the loader's search for the multiplying side.  One ring for the block: every wavefront writes the
  // same values and may read what another wrote.  What keeps an entry until the slowest has read it is the barrier of each half-step: with
  // three half-steps or more per tile no wavefront has opened a tile past n + 3 while another still fetches the entry of n + 1.
  __shared__ __attribute__((aligned(16))) int s_tile[4][4];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave >> 1, wn = wave & 1;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int uwm = uwave >> 1, uwn = uwave & 1;
  const int G = gridDim.x;
  // Blocks b, b + 8, ... share an XCD and get consecutive tiles.  In the last, partial round of a launch with two blocks per
  // compute unit (b and b + G / 2) the first G / 2 positions are one block of every compute unit, again XCD by XCD.
  const int xcd = (int)blockIdx.x & 7, in_xcd = (int)blockIdx.x >> 3, cu_xcd = (G / S::BLOCKS) >> 3;
  const int full_pos = xcd * (G >> 3) + in_xcd;
  const int part_pos = (in_xcd / cu_xcd) * (G / S::BLOCKS) + xcd * cu_xcd + in_xcd % cu_xcd;
  const int nh = (a.K + HK - 1) / HK;

  const bool probe = a.clock_probe && blockIdx.x < MAX_STREAM_GRID;
  const unsigned long long probe_c0 = probe ? clock64() : 0ull, probe_t0 = probe ? wall_clock64() : 0ull;
  for (int i = threadIdx.x; i <= a.E; i += NTHREADS) s_off[i] = a.offsets ? a.offsets[i] : a.Tk / a.E * i;
  __syncthreads();

  const TilePlan plan = plan_tiles<S>(s_off, a.E, tiles_n, nh, G, STATIC4, ACT == 0 && a.tail_ws != nullptr, lane);
  // This block's part of the last, partial round: tile number (-1: none), chunk of its contraction, index of the fp32
  // partial tile it leaves (-1: the tile is whole).
  int last_tile = -1, last_h0 = 0, last_hn = nh, last_part = -1;
  if (part_pos < plan.whole) {
    last_tile = plan.rounds * G + part_pos;
  } else if (part_pos - plan.whole < plan.rest * plan.split) {
    const int u = part_pos - plan.whole, chunk = u % plan.split;
    last_tile = plan.rounds * G + plan.whole + u / plan.split;
    if (plan.split > 1) {
      last_h0 = chunk * plan.chunk;
      last_hn = min(nh, last_h0 + plan.chunk) - last_h0;
      last_part = u;
    }
  }
  const int rounds = plan.rounds, m_tiles = plan.m_tiles;
  // Arguments needed once per tile are read from the kernel's argument segment again where they are used: kept in scalar
  // registers they would not fit beside the loader's state, and the loop would fetch spilled registers every half-step.
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
    const int w = seq < rounds ? seq * G + full_pos : last_tile;
    int mt, nt, e, row0, row_end;
    tile_coords(w, m_tiles, tiles_n, group_m, mt, nt);
    locate_rows<S::TM>(s_off, a.E, mt, lane, e, row0, row_end);
    t.seq = seq;
    t.e = __builtin_amdgcn_readfirstlane(e);
    t.row0 = __builtin_amdgcn_readfirstlane(row0);
    t.row_end = __builtin_amdgcn_readfirstlane(row_end);
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
  auto half_steps = [&](const Tile &t) { return t.seq < rounds ? nh : last_hn; };
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

  S2SOps<S, TRANS_W, KTAIL> ops;
  ops.uwave = uwave;
  ops.b_step = TRANS_W ? (uint32_t)(HK * 2) : (uint32_t)(HK * 2) * (uint32_t)a.ldw;
  ops.last = nh - 1;
  auto setup_sources = [&](const Tile &t) {
    const auto p = args();
    const int K = p->K, N = p->N;
    const uint32_t row_bytes = (uint32_t)K * 2u, ldw_bytes = (uint32_t)p->ldw * 2u;
    const bool gathered = p->a_map.o != nullptr;
    // gathered rows are addressed from the start of A, expert-sorted rows from the tile's first row
    const bool second = DENSE_PAIR && p->C2 && t.e == 1;
    ops.win_a = buffer_window((const bf16_t *)(second ? p->A2 : p->A) + (gathered ? 0 : (size_t)t.row0 * K),
                              (uint32_t)(gathered ? p->Tk / p->a_map.fan : min(S::TM, t.row_end - t.row0)) * row_bytes);
    ops.win_b = buffer_window((const bf16_t *)(second ? p->W2 : p->W) + (size_t)t.e * p->w_stride, (uint32_t)(TRANS_W ? N : K) * ldw_bytes);
    if (S::ONCE) ops.again = t.row_end - __builtin_amdgcn_readfirstlane(s_off[t.e]) - S::TM;
    const int *idx = &s_idx[t.seq & 3][0];
#pragma unroll
    for (int I = 0; I < S::NLA; ++I) {
      const int r = (wave * S::NLA + I) * 16 + (lane >> 2), c = (lane & 3) ^ kc_swz(r);
      uint32_t src = (uint32_t)r;
      if (gathered) {
        const uint32_t slot = (uint32_t)idx[r];
        src = magic_a ? __umulhi(slot, magic_a) : slot;
      }
      ops.oa[I] = src * row_bytes + (uint32_t)c * 16u;
      if (KTAIL) ops.ta[I] = (nh - 1) * HK + c * 8 >= K ? ~0u : 0u;
    }
#pragma unroll
    for (int I = 0; I < NLD; ++I) {
      int r, c;
      if (TRANS_W) {
        kc_lane_slot(wave, lane, I, r, c);
        ops.ob[I] = (uint32_t)min(t.n0 + r, N - 1) * ldw_bytes + (uint32_t)c * 16u;
        if (KTAIL) ops.tb[I] = (nh - 1) * HK + c * 8 >= K ? ~0u : 0u;
      } else {
        tr_lane_slot(wave, lane, I, r, c);
        int col = t.n0 + c * 8;
        if (SWIGLU) {
          // tile column v = c * 8: wavefront column half v / 128 takes 64 gate columns then their 64 up columns
          const int v = c * 8, w = v & 127, gate = t.n0 + (v >> 7) * 64 + (w & 63);
          col = (gate < N / 2) ? gate + (w >> 6) * (N / 2) : N;
        }
        if (col >= N) col = 0;
        ops.ob[I] = (uint32_t)r * ldw_bytes + (uint32_t)col * 2u;
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
  int step_end = ops.step + half_steps(lt);
  bool loader_live = true;
  // loader moves one half-step on; at a tile end it opens the upcoming tile and requests the rows of the one after
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
    step_end = ops.step + half_steps(lt);
    have_upcoming = next_tile(upcoming);
    if (have_upcoming) fetch_rows(upcoming);
    setup_sources(lt);
  };

  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
#pragma unroll 1
  for (int st = 0; st < S::SLOTS - 1; ++st) {
#pragma unroll
    for (int I = 0; I < S::NL; ++I) ops.load(I, lds0 + st * S::SLOT_BYTES);
    advance_loader();
  }
#pragma unroll
  for (int I = 0; I < S::HALF; ++I) ops.load(I, lds0 + (S::SLOTS - 1) * S::SLOT_BYTES);
  wait_loads<S::IN_FLIGHT + S::HALF>();   // the first stage has landed
  __syncthreads();
  f32x16 acc[S::FM][FR];
  Frags<S> f0, f1;
#pragma unroll
  for (int g = 0; g < 3; ++g) read_frag_group<S>(ops, f0, smem, 0, g, wm, wn, lane);

  uint32_t cur = 0;            // LDS slot of the half-step at hand (0 at every tile start with STATIC4)
  // One half-step in slot `slot`.  `relaxed`: an epilogue's stores were issued after the loads this wait is for.
  auto half_step = [&](auto first, auto last, uint32_t slot, bool relaxed) {
    constexpr bool GO_ON = !(decltype(last)::value && S::PATCH_IN_SLOT);
    phase<0, decltype(first)::value, true, true, S>(ops, f0, f1, smem + slot, lds0 + Ring<S>::before(slot), wm, wn, lane, acc);
    advance_loader();
    if (relaxed) middle<S, STORES>(); else middle<S, 0>();
    phase<1, false, GO_ON, GO_ON, S>(ops, f1, f0, smem + Ring<S>::after(slot), lds0 + slot, wm, wn, lane, acc);
  };
  using No = std::false_type;
  using Yes = std::true_type;
  for (;;) {   // one tile per trip
    // stores of the previous tile's epilogue lie behind the loads that the first SLOTS - 2 waits are for
    const bool stored = ct.seq > 0;
    const int hn = half_steps(ct);
    if constexpr (STATIC4) {
      half_step(Yes{}, No{}, 0 * S::SLOT_BYTES, stored);
      half_step(No{}, No{}, 1 * S::SLOT_BYTES, stored);
      half_step(No{}, No{}, 2 * S::SLOT_BYTES, false);
      half_step(No{}, No{}, 3 * S::SLOT_BYTES, false);
      for (int h = 4; h < hn; h += 4) {
        half_step(No{}, No{}, 0 * S::SLOT_BYTES, false);
        half_step(No{}, No{}, 1 * S::SLOT_BYTES, false);
        half_step(No{}, No{}, 2 * S::SLOT_BYTES, false);
        half_step(No{}, No{}, 3 * S::SLOT_BYTES, false);
      }
    } else {
      half_step(Yes{}, No{}, cur, stored);
      cur = Ring<S>::after(cur);
      for (int h = 1; h < hn - 1; ++h) {
        half_step(No{}, No{}, cur, stored && h < S::SLOTS - 2);
        cur = Ring<S>::after(cur);
      }
      half_step(No{}, Yes{}, cur, false);
    }
    const int lane = ACT == 6 ? lane_here(threadIdx.x & 63) : (int)(threadIdx.x & 63);
    char *patch = S::PATCH_IN_SLOT ? smem + cur + S::A_BYTES + uwave * EPI_WAVE_BYTES
                                   : smem + S::SLOTS * S::SLOT_BYTES + uwave * EPI_WAVE_BYTES;
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
      const int gcol = ct.n0 + uwn * (TB / 2), ldc = ACT == 3 ? 2 * N : N;
      const uint32_t slot_bytes = (uint32_t)p->Tk * (uint32_t)N * 2u;                 // ACT 6: of dH and of H
      const window_t win_c = ACT == 6 ? make_window(p->C, slot_bytes) : sorted_window(p->C, ldc, 2);
      BwdRows b;
      b.saved = ACT == 6 ? make_window(p->H_in, slot_bytes) : sorted_window(ACT == 3 ? p->Hpre_in : p->H_in, ldc, 2);
      b.places = &s_idx[ct.seq & 3][uwm * (S::TM / 2)];
      b.left = left;
      b.saved_bytes = (uint32_t)ldc * 2u;
      b.scale = sorted_window(p->row_scale, 1, 4);
      b.dp = sorted_window(p->dp_part, 2 * tiles_n, 4);
      b.part_bytes = (uint32_t)tiles_n * 8u;
      b.part_col = (uint32_t)(ct.n0 / TB) * 2u + uwn;
      b.n = N;
      b.gcol = gcol;
      if constexpr (ACT == 3) {
        store_wave_tile_swiglu_bwd<S::BLOCKS == 1>(
            acc, patch, b,
            [&](int fm, int half, int up) { return sorted_block(win_c, ldc, fm, up * N + gcol + half * 64, N - gcol - half * 64); }, lane);
      } else {
        const window_t win_w = ACT >= 5 ? sorted_window(p->Hw_out, N, 2) : win_c;
        auto dest = [&](int fm, int half) {
          if constexpr (ACT == 6) return slot_block(win_c, N, b.places, left, fm, gcol + half * 64);
          else return sorted_block(win_c, ldc, fm, gcol + half * 64, N - gcol - half * 64);
        };
        store_wave_tile_dp<S::BLOCKS == 1, ACT >= 5, ACT == 6>(
            acc, patch, b, dest,
            [&](int fm, int half) { return sorted_block(win_w, N, fm, gcol + half * 64, N - gcol - half * 64); },
            lane);
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
    if constexpr (S::PATCH_IN_SLOT) {   // what the last phase B held back
#pragma unroll
      for (int I = 0; I < S::HALF; ++I) ops.load(I, lds0 + cur);
#pragma unroll
      for (int g = 0; g < 3; ++g) read_frag_group<S>(ops, f0, smem + Ring<S>::after(cur), 0, g, wm, wn, lane);
    }
    if constexpr (!STATIC4) cur = Ring<S>::after(cur);
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
__global__ void __launch_bounds__(256) s2s_tail_reduce_kernel(S2SArgs a, int tiles_n, int group_m, int G, int static4) {
  __shared__ int s_off[MAX_E + 1];
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i <= a.E; i += 256) s_off[i] = a.offsets ? a.offsets[i] : a.Tk / a.E * i;
  __syncthreads();
  const TilePlan plan = plan_tiles<S>(s_off, a.E, tiles_n, (a.K + HK - 1) / HK, G, static4 != 0, true, lane);
  if (plan.split <= 1) return;
  constexpr int PER_SLICE = S::PART / 4 / TAIL_SLICES;
  for (int unit = blockIdx.x; unit < plan.rest * TAIL_SLICES; unit += TAIL_BLOCKS) {
    const int tile = unit / TAIL_SLICES, slice = unit % TAIL_SLICES;
    int mt, nt, e, row0, row_end;
    tile_coords(plan.rounds * G + plan.whole + tile, plan.m_tiles, tiles_n, group_m, mt, nt);
    locate_rows<S::TM>(s_off, a.E, mt, lane, e, row0, row_end);
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
// groupXTY, persistent: dW[e] = Xbar_e^T dYbar_e over expert-sorted rows (Alg. 2 groups both
// operands first; gathering the token rows inside this kernel measured a third slower than a
// `group` copy followed by this kernel, the same ranking the paper reports).
// ======================================================================================
// The loader cursor runs three slots ahead of the multiplying cursor over the same slot
// sequence: the half-steps of a tile rounded up to a multiple of four (at least four) slots,
// tiles in largest-expert-first order.  Slots past a segment's end load a block of zeros, so a
// tile of an empty expert multiplies zeros and writes zeros.
struct DWCursor {
  int seq;        // position in this block's tile list
  int step, ns;   // slot within the tile, slots of the tile
  int nh;         // half-steps (0 for an empty expert)
  int e, lo, hi, m0, n0;
  bool further;   // a tile of dW3
  bool live;
};

struct DWStreamOps {
  int ra[NLD], ka[NLD];      // per load instruction: contraction row within a slot, 16-byte column chunk
  int uwave;
  // The loader's current group of four slots: range-checked windows that start at the group's first
  // row and end with the expert's segment (rows past it, padded slots and empty experts read zeros and
  // add nothing to the sum), per-lane byte offsets of the tile's columns inside a slot, and the byte
  // offset of the current slot inside the group.
  int32x4 win_a, win_b;
  uint32_t oa[NLD], ob[NLD];
  uint32_t sub_a, sub_b;
  __device__ __forceinline__ void load(int I, uint32_t slot_lds) const {
    load16_to_lds_checked(I < NLD ? win_a : win_b, I < NLD ? oa[I] + sub_a : ob[I - NLD] + sub_b,
                          slot_lds + (I / NLD) * TILE_BYTES + inst_off(uwave, I % NLD));
  }
  __device__ __forceinline__ bf16x8 frag_a(const char *tile, int base, int kk, int l) const { return tr_frag(tile, base, kk, l); }
  __device__ __forceinline__ bf16x8 frag_b(const char *tile, int base, int kk, int l) const { return tr_frag(tile, base, kk, l); }
};

// tile number inside an expert -> first row and column of the tile: bands of group_m M-tiles, N-tile by
// N-tile, so that the 32 consecutive tiles an XCD holds at a time form a compact patch sharing few panels
__device__ __forceinline__ void dw_tile_origin(int t, int tiles_m, int tiles_n, int &m0, int &n0) {
  const int group_m = (tiles_m % 8 == 0) ? 8 : ((tiles_m % 4 == 0) ? 4 : ((tiles_m % 2 == 0) ? 2 : 1));
  const int band = t / (group_m * tiles_n), r = t - band * (group_m * tiles_n);
  m0 = (band * group_m + r % group_m) * TB;
  n0 = (r / group_m) * TB;
}
// rows of chunk `chunk` of `split` of the segment [lo, hi): chunks are whole groups of four half-steps
__device__ __forceinline__ void dw_chunk_rows(int lo, int hi, int split, int chunk, int &clo, int &chi) {
  const int nh = (hi - lo + HK - 1) / HK;
  const int len = (((nh + split - 1) / split + 3) & ~3) * HK;
  clo = min(hi, lo + chunk * len);
  chi = min(hi, clo + len);
}

// split > 1 (only when all experts' tiles times split fit one round of the grid): unit T is chunk T % split of
// tile T / split, experts in their own order, and the result is an fp32 partial tile number T in a.split_ws.
// KIND (kernels of their own: the choice of operands sits in every slot): DW_PAIR segment 1 is the second weight gradient of DWArgs;
// DW_TWO every expert's tiles are followed by those of its dW3.
enum { DW_ONE = 0, DW_PAIR = 1, DW_TWO = 2 };
template <int KIND> __global__ void __launch_bounds__(NTHREADS, 1) dw_stream_kernel(DWArgs a, int tiles_m, int tiles_n, int split) {
  constexpr bool DENSE_PAIR = KIND == DW_PAIR;
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

  auto open_tile = [&](DWCursor &c, int seq) {
    c.seq = seq;
    const int U = seq * G + slot_in_round;
    const int T = U / split;
    int rank = T / per_expert;
    c.live = rank < a.E && (split == 1 || seq == 0);
    if (!c.live) return;
    int t = T - rank * per_expert;
    c.e = split > 1 ? rank : __builtin_amdgcn_readfirstlane(s_order[rank]);   // LDS reads land in vector registers: make them scalar again
    c.lo = __builtin_amdgcn_readfirstlane(s_off[c.e]);
    c.hi = __builtin_amdgcn_readfirstlane(s_off[c.e + 1]);
    if (split > 1) dw_chunk_rows(c.lo, c.hi, split, U - T * split, c.lo, c.hi);
    c.further = KIND == DW_TWO && t >= per_first;
    if (c.further) dw_tile_origin(t - per_first, tiles_m3, tiles_n3, c.m0, c.n0);
    else dw_tile_origin(t, tiles_m, tiles_n, c.m0, c.n0);
    c.nh = (c.hi - c.lo + HK - 1) / HK;
    // Slots come in groups of four so that every tile starts in LDS stage 0 and the loop can be written
    // with compile-time stages; the up to three extra slots (four for an empty expert) load the zero
    // block and add nothing.
    c.ns = max((c.nh + 3) & ~3, 4);
    c.step = 0;
  };
  auto advance = [&](DWCursor &c) {
    if (!c.live) return;
    if (++c.step < c.ns) return;
    // keeps the tile lookup behind this (rarely taken) branch: without it the compiler evaluates
    // the lookup's integer divisions in every half-step and selects the results
    __asm__ volatile("" ::: "memory");
    open_tile(c, c.seq + 1);
  };

  DWStreamOps ops;
  ops.uwave = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
  for (int I = 0; I < NLD; ++I) tr_lane_slot(wave, lane, I, ops.ra[I], ops.ka[I]);
  const bf16_t *A = (const bf16_t *)a.A, *B = (const bf16_t *)a.B;
  // loader cursor: publish the slot whose eight loads are issued next
  int shown_m0 = -1, shown_n0 = -1, shown_further = -1;
  auto resolve = [&](const DWCursor &c) {
    const int first = c.lo + (c.step & ~3) * HK;                 // first row of this group of four slots
    const int left = c.live ? max(c.hi - first, 0) : 0;          // rows of the segment from there on
    const int base_row = left > 0 ? first : 0;
    const unsigned long long cap = 0xffffffffull;
    const bool second = DENSE_PAIR && c.e == 1, further = KIND == DW_TWO && c.further;
    const int M = further ? a.M3 : a.M, N = further ? a.N3 : a.N;
    const uint32_t row_a = (uint32_t)M * 2u, row_b = (uint32_t)N * 2u;   // bytes per operand row
    ops.win_a = buffer_window((further ? (const bf16_t *)a.A3 : second ? (const bf16_t *)a.A2 : A) + (size_t)base_row * M, (uint32_t)min((unsigned long long)left * row_a, cap));
    ops.win_b = buffer_window((further ? (const bf16_t *)a.B3 : second ? (const bf16_t *)a.B2 : B) + (size_t)base_row * N, (uint32_t)min((unsigned long long)left * row_b, cap));
    ops.sub_a = (uint32_t)(c.step & 3) * HK * row_a;
    ops.sub_b = (uint32_t)(c.step & 3) * HK * row_b;
    if (c.m0 != shown_m0 || c.n0 != shown_n0 || (KIND == DW_TWO && (int)c.further != shown_further)) {   // a new tile: its columns' offsets inside a slot
      shown_m0 = c.m0;
      shown_n0 = c.n0;
      shown_further = c.further;
#pragma unroll
      for (int J = 0; J < NLD; ++J) {
        int ca = c.m0 + ops.ka[J] * 8, cb = c.n0 + ops.ka[J] * 8;
        if (ca >= M) ca = 0;
        if (cb >= N) cb = 0;
        ops.oa[J] = (uint32_t)ops.ra[J] * row_a + (uint32_t)ca * 2u;
        ops.ob[J] = (uint32_t)ops.ra[J] * row_b + (uint32_t)cb * 2u;
      }
    }
  };

  DWCursor cc, lc;
  open_tile(cc, 0);
  if (!cc.live) return;
  lc = cc;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
  char *patch = smem + Big::SLOTS * Big::SLOT_BYTES + ops.uwave * EPI_WAVE_BYTES;
#pragma unroll 1
  for (int st = 0; st < Big::SLOTS - 1; ++st) {
    resolve(lc);
#pragma unroll
    for (int I = 0; I < Big::NL; ++I) ops.load(I, lds0 + st * Big::SLOT_BYTES);
    advance(lc);
  }
  resolve(lc);
#pragma unroll
  for (int I = 0; I < Big::HALF; ++I) ops.load(I, lds0 + (Big::SLOTS - 1) * Big::SLOT_BYTES);
  wait_loads<Big::IN_FLIGHT + Big::HALF>();
  __syncthreads();
  Frags<Big> f0, f1;
  f32x16 acc[FR][FR];
#pragma unroll
  for (int g = 0; g < 3; ++g) read_frag_group<Big>(ops, f0, smem, 0, g, wm, wn, lane);

  auto half_step = [&](auto first, auto slot_c, bool relaxed) {
    constexpr uint32_t SLOT = decltype(slot_c)::value * Big::SLOT_BYTES;
    phase<0, decltype(first)::value, true, true, Big>(ops, f0, f1, smem + SLOT, lds0 + Ring<Big>::before(SLOT), wm, wn, lane, acc);
    advance(lc);
    resolve(lc);
    if (relaxed) middle<Big, EpilogueStores<Big::FM, 0>>(); else middle<Big, 0>();
    phase<1, false, true, true, Big>(ops, f1, f0, smem + Ring<Big>::after(SLOT), lds0 + SLOT, wm, wn, lane, acc);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  for (;;) {   // one tile per trip
    const bool stored = cc.seq > 0;
    half_step(std::true_type{}, I0{}, stored);
    half_step(std::false_type{}, I1{}, stored);
    half_step(std::false_type{}, I2{}, false);
    half_step(std::false_type{}, I3{}, false);
    for (int h = 4; h < cc.ns; h += 4) {
      half_step(std::false_type{}, I0{}, false);
      half_step(std::false_type{}, I1{}, false);
      half_step(std::false_type{}, I2{}, false);
      half_step(std::false_type{}, I3{}, false);
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
    open_tile(cc, cc.seq + 1);
    if (!cc.live) break;
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

template <typename S, bool TRANS_W, bool SCATTER_OUT, int ACT, bool STATIC4, bool WIDE> int launch_s2s_one(hipStream_t s, const S2SArgs &a) {
  const int tiles_n = (ACT == 1 || ACT == 2) ? ceil_div(a.N / 2, TB / 2) : ceil_div(a.N, TB);
  const long long tiles_m = ceil_div(a.Tk, S::TM) + a.E;     // upper bound on sum_e ceil(n_e / TM)
  const int group_m = a.group_m * (TB / S::TM), grid = a.grid * S::BLOCKS;
  if (tiles_m * tiles_n > 0x7fffffffLL) return SMOE_ERR_UNSUPPORTED;
  S2SArgs args = a;
  int chunk;
  if (ACT != 0 || choose_split(ceil_div(a.K, HK), 4, STATIC4, chunk) == 1) args.tail_ws = nullptr;   // too short to pay: no second kernel
  hipLaunchKernelGGL((s2s_stream_kernel<S, TRANS_W, SCATTER_OUT, ACT, STATIC4, WIDE>), dim3(grid), dim3(NTHREADS), S::LDS_BYTES, s, args,
                     tiles_n, group_m, division_magic(a.a_map.o ? a.a_map.fan : 1));
  SMOE_LAUNCH_CHECK();
  if (args.tail_ws) {   // adds and stores the partial tiles of a split last round (no-op when nothing was split)
    hipLaunchKernelGGL((s2s_tail_reduce_kernel<S, SCATTER_OUT>), dim3(TAIL_BLOCKS), dim3(256), 0, s, a, tiles_n, group_m, grid, STATIC4 ? 1 : 0);
    SMOE_LAUNCH_CHECK();
  }
  return SMOE_OK;
}
// Which shape a launch takes.  The row counts are on the device, so an expert is taken to have r = Tk / E rows: r / TM + 1/2
// tiles on average, one when it has few rows.  Estimated time in microseconds:
//   a half-step: 0.85 (Big), 1.03 for two pair tiles sharing a compute unit, 0.5 for one alone; epilogue and tile set-up 6 / 6 / 4;
//   a split's partial tiles: written and read at 4.5 TB/s, and 5 for the second kernel.
// Many rounds of long contractions are the Big tile's (they run at the package's power limit, and the pair's operand traffic
// costs power), so the pair is only asked where it measured faster: contractions up to 2048, or up to 6144 with little more
// than two pair tiles per compute unit, and not for an estimated gain under 5 % (at 1 % it lost as often as it won).  Measured, Big / Pair in us:
//   8192 rows, 8 experts: 1024 -> 5632 with SwiGLU 120 / 108, 2816 -> 1024 77 / 75, its W1^T counterpart (5632 -> 1024) 160 / 140;
//   6216 rows, 64 experts: 2048 -> 1024 with SwiGLU 63 / 52, 512 -> 2048 36 / 28;  8192 rows, 1 expert: 2048 -> 1024 62 / 42;
//   32768 rows, 8 experts: 1024 -> 5632 372 / 393, 5632 -> 1024 400 / 458;  65536 rows, 64 experts: 2048 -> 1024 286 / 308;
//   2048 rows, 8 experts: 4096 -> 28672 590 / 810;  4096 rows, 8 experts: 4096 -> 8192 320 / 340.
template <typename S> float launch_estimate(const S2SArgs &a, int tiles_n, bool static4, bool may_split, long long &total) {
  const float rows = (float)a.Tk / a.E;
  const int nh = ceil_div(a.K, HK), G = a.grid * S::BLOCKS;
  const float m_tiles = a.E == 1 || a.C2 ? (float)a.E * ceil_div(a.Tk / a.E, S::TM) : (rows >= S::TM ? rows / S::TM + 0.5f : 1.0f) * (a.Tk < a.E ? a.Tk : a.E);
  total = (long long)(m_tiles * tiles_n + 0.5f);
  const float full = (S::BLOCKS == 1 ? 0.85f : 1.03f) * nh + 6.f, one = S::BLOCKS == 1 ? full : 0.5f * nh + 4.f;
  const int rem = (int)(total % G), whole = S::BLOCKS > 1 && rem > a.grid ? a.grid : 0, rest = rem - whole;
  float t = (total / G) * full;
  int chunk = nh, split = 1;
  if (may_split && rest > 0) split = choose_split(nh, (whole ? a.grid : G) / rest, static4, chunk);
  const bool crowded = rest * split > a.grid;     // some compute unit has two blocks in the last round
  if (whole) t += split > 1 ? one + (full - one) / split : (rest ? full : one);
  else if (rest) t += (crowded ? full : one) / split;
  if (split > 1) t += 5.f + rest * split * (S::PART * 8.f / 4.5e6f);
  return t;
}
bool prefer_pair(const S2SArgs &a, int tiles_n, bool may_split) {
  long long big, pair;
  const float t_big = launch_estimate<Big>(a, tiles_n, a.K % (4 * HK) == 0, may_split, big);
  const float t_pair = launch_estimate<Pair>(a, tiles_n, false, may_split, pair);
  return (a.K <= 2048 || (a.K <= 6144 && pair * 4 <= a.grid * 9LL)) && t_pair < 0.95f * t_big;
}
template <bool TRANS_W, bool SCATTER_OUT, int ACT = 0> int launch_s2s_cfg(hipStream_t s, const S2SArgs &a) {
  const bool static4 = a.K % (4 * HK) == 0;
  if constexpr (SCATTER_OUT && ACT == 0)
    if ((long long)a.Tk * a.N * 2 > 0xfffffff0LL) {   // rows a 32-bit offset does not reach
      if (static4) return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, true, true>(s, a);
      return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, false, true>(s, a);
    }
  // The epilogue of ACT 6 (two offsets per row, two outputs) does not fit the 128 registers of a pair: 72 of them spilled, and the
  // product of 32768 rows, 2048 -> 512, took 225 us of 121.
  if constexpr (ACT != 6) {
    const int tiles_n = (ACT == 1 || ACT == 2) ? ceil_div(a.N / 2, TB / 2) : ceil_div(a.N, TB);
    const bool may_split = ACT == 0 && a.tail_ws;
    if (a.tile_shape == 1 || (a.tile_shape == 0 && prefer_pair(a, tiles_n, may_split))) {
      // At most one tile row per expert on average: most of W is read once, and where the call's weights exceed the last-level cache
      // keeping its lines only pushes other data out (6216 rows, 64 experts: 2048 -> 2 x 512 in 60 us, past the caches 53).  With
      // reuse they belong there (8192 rows and 8 experts, 1024 -> 5632: 113 us, past the caches 156), so a tile of an expert that has
      // several takes them the ordinary way (777 tokens on 64 experts with Zipf(1.2) loads, 2048 -> 2 x 512 -> 2048: the forward pass
      // 133 us with all of W past the caches, 129 with none, 125 so).
      if constexpr (!TRANS_W)
        if ((long long)a.Tk <= (long long)a.E * Pair::TM && weights_pass_caches(a))
          return launch_s2s_one<PairOnce, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
      return launch_s2s_one<Pair, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
    }
  }
  if (static4) return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, true, false>(s, a);
  return launch_s2s_one<Big, TRANS_W, SCATTER_OUT, ACT, false, false>(s, a);
}

int launch_dw_stream_impl(hipStream_t s, const DWArgs &a) {
  int tiles_m = ceil_div(a.M, TB), tiles_n = ceil_div(a.N, TB);
  // Row split: only when every tile of every expert, times the split, fits one round of the grid, and only when
  // it shortens the contraction by more than the partial tiles cost (as for the split last round above).
  int split = 1;
  const long long tiles = (long long)a.E * tiles_m * tiles_n;
  if (a.split_ws && tiles * 2 <= a.grid) {
    const long long nh = a.Tk / a.E / HK;            // half-steps of an average segment
    split = (int)(a.grid / tiles < 8 ? a.grid / tiles : 8);
    if (nh - nh / split < SPLIT_MIN_SAVED) split = 1;
  }
  if (a.dW3) split = 1;
  if (a.dW3) hipLaunchKernelGGL(dw_stream_kernel<DW_TWO>, dim3(a.grid), dim3(NTHREADS), Big::LDS_BYTES, s, a, tiles_m, tiles_n, split);
  else if (a.dW2) hipLaunchKernelGGL(dw_stream_kernel<DW_PAIR>, dim3(a.grid), dim3(NTHREADS), Big::LDS_BYTES, s, a, tiles_m, tiles_n, split);
  else hipLaunchKernelGGL(dw_stream_kernel<DW_ONE>, dim3(a.grid), dim3(NTHREADS), Big::LDS_BYTES, s, a, tiles_m, tiles_n, split);
  SMOE_LAUNCH_CHECK();
  if (split > 1) {
    hipLaunchKernelGGL(dw_split_reduce_kernel, dim3((unsigned)tiles, TAIL_SLICES), dim3(256), 0, s, a, tiles_m, tiles_n, split);
    SMOE_LAUNCH_CHECK();
  }
  return SMOE_OK;
}
}  // namespace

// A tile must have at least three half-steps (the index ring assumes it); the expert offsets must fit their LDS cache; order
// indices are divided by the fan-out with a multiply-high that is exact while Tk * fan < 2^32.  Every source offset (from
// the start of a gathered A, of an expert's matrix, of a tile's first row) must fit 32 bits with the last half-step's
// overhang, and a tile's rows of an output 31 bits.
bool s2s_stream_supported(const S2SArgs &a) {
  const long long fan = a.a_map.o ? a.a_map.fan : 1;
  const long long a_rows = a.a_map.o ? (long long)a.Tk / fan + 1 : TB;
  const long long w_rows = a.trans_w ? a.N : a.K;
  return a.grid >= 8 && a.grid % 8 == 0 && a.grid <= MAX_STREAM_GRID && a.group_m >= 1 && a.K % 8 == 0 && a.K > 2 * HK && a.N % 8 == 0 &&
         a.ldw % 8 == 0 && a.Tk > 0 && a.E <= MAX_E && (long long)a.Tk * fan < 0x100000000LL && (a_rows * a.K + HK) * 2 < 0x100000000LL &&
         (w_rows + HK) * a.ldw * 2 < 0x100000000LL && (long long)TB * a.N * 4 < 0x80000000LL;
}
bool s2s_stream_swiglu_bwd_supported(const S2SArgs &a) {
  return s2s_stream_supported(a) && a.trans_w && !a.c_map.o && a.Hpre_in && a.row_scale && a.dp_part && a.N % 8 == 0;
}

bool s2s_stream_dp_supported(const S2SArgs &a) {
  const bool slots_fit = !a.c_map.o || (a.Hw_out && (long long)a.Tk * a.N * 2 <= 0xfffffff0LL);   // ACT 6: 32-bit offsets of slot rows
  return s2s_stream_supported(a) && a.trans_w && slots_fit && a.H_in && !a.Hpre_in && a.row_scale && a.dp_part && a.N % 8 == 0;
}

bool s2s_stream_swiglu_supported(const S2SArgs &a) {
  return s2s_stream_supported(a) && !a.trans_w && !a.c_map.o && a.H && a.N % 16 == 0;
}

int launch_s2s_stream(hipStream_t s, const S2SArgs &a) {
  const bool scatter_out = a.c_map.o != nullptr;
  if (a.dp_part && a.Hpre_in) {
    if (!s2s_stream_swiglu_bwd_supported(a)) return SMOE_ERR_UNSUPPORTED;
    return launch_s2s_cfg<true, false, 3>(s, a);
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

bool dw_stream_supported(const DWArgs &a) {
  long long tiles = (long long)a.E * ((long long)ceil_div(a.M, TB) * ceil_div(a.N, TB) + (long long)ceil_div(a.M3, TB) * ceil_div(a.N3, TB));
  return a.M % 8 == 0 && a.N % 8 == 0 && a.M3 % 8 == 0 && a.N3 % 8 == 0 && a.Tk > 0 && a.E <= MAX_E && tiles + MAX_STREAM_GRID < 0x7fffffffLL && a.grid >= 8 &&
         a.grid % 8 == 0 && a.grid <= MAX_STREAM_GRID && (long long)TB * a.N * 2 < 0x80000000LL && (long long)TB * a.N3 * 2 < 0x80000000LL;
}

// Together two weight gradients save the rounds that their last tiles fill only in part, and a launch, while a slot costs 3 % more
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
  if constexpr (ACT != 6)
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<Pair, TRANS_W, SCATTER_OUT, ACT, false, false>, Pair::LDS_BYTES);
  if constexpr (!TRANS_W)
    if (rc == SMOE_OK) rc = set_lds_limit(s2s_stream_kernel<PairOnce, TRANS_W, SCATTER_OUT, ACT, false, false>, Pair::LDS_BYTES);
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
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_ONE>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_PAIR>, Big::LDS_BYTES);
  if (rc == SMOE_OK) rc = set_lds_limit(dw_stream_kernel<DW_TWO>, Big::LDS_BYTES);
  return rc;
}
