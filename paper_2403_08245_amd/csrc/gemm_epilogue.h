// Epilogues of the persistent matrix-core kernels: a wavefront's accumulators -> bf16 -> LDS patch -> whole-line
// stores, with the activation, its derivative or the routing-weight gradient folded in.  A wavefront's tile is
// FM x 4 fragments of 32 x 32 (FM = 4 in the 256 x 256 kernels, 2 in the 128 x 256 ones).
//
// Global accesses go through raw buffer windows: an address is one 32-bit lane offset (usually a loop-invariant lane part
// plus a scalar), and rows past the segment or columns past the width are switched off by an offset outside the window
// instead of a branch or a select of 64-bit pointers.  With one wavefront per SIMD every instruction of an epilogue is
// time the matrix cores idle.  Every store is issued unconditionally, so a wavefront's stores per tile are a constant
// that the kernels' load waits can step over (EpilogueStores).
#pragma once
#include "mfma_common.h"

namespace {

constexpr int EPI_WAVE_BYTES = 32 * 128;   // one wavefront's patch: 32 rows of 64 bf16 columns

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t window_t;
constexpr uint32_t OFF_WINDOW = 0x80000000u;   // a lane offset no window reaches (windows are shorter than 2 GB where it is added to)
__device__ __forceinline__ window_t make_window(const void *base, uint32_t bytes) {
  const unsigned long long p = (unsigned long long)base;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void *)(((unsigned long long)hi << 32) | lo), 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// Moves one accumulator element out of the accumulation register file right where it is
// used.  Left to itself the register allocator copies all accumulators of a lane into
// ordinary registers at the top of the epilogue, which cannot fit beside the operand
// fragments and load addresses that stay live for the next tile.
__device__ __forceinline__ float acc_read(float a) {
  float v;
  __asm__ volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}
// the last matrix instructions must have retired before their results are read by hand
__device__ __forceinline__ void acc_settle() { __asm__ volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// ---- the LDS patch as a pipeline ------------------------------------------------------------------------
// A 32 x 64 block of bf16 results goes accumulator layout -> patch (8-byte writes, a lane's 4 consecutive columns)
// -> whole rows back out (16-byte reads, eight lanes per 128-byte row) -> global memory.  LDS operations of one
// wavefront execute in order, so the block's row reads may be issued right behind its writes and the next block's
// writes right behind those reads, with no wait in between; only the global stores need the read data.  The
// stores of block n are therefore issued after block n+1 has been written and read: the LDS latency of one block
// hides behind the accumulator reads and conversions of the next one instead of being sat out four times per block.
// The patch has no padding; its 16-byte chunks are rotated by the row (chunk ^ row % 8), which keeps both the 8-byte
// writes (32 rows, one chunk) and the 16-byte reads (whole rows) free of bank conflicts.
__device__ __forceinline__ char *patch_slot(char *patch, int row, int chunk) { return patch + row * 128 + ((chunk ^ (row & 7)) << 4); }
// where a lane's four columns 8 * g + 4 * (lane / 32) of fragment half f2 go (its own row is lane % 32)
__device__ __forceinline__ void patch_put(char *patch, int lane, int f2, int g, bf16x4 v) {
  *reinterpret_cast<bf16x4 *>(patch_slot(patch, lane & 31, f2 * 4 + g) + 8 * (lane >> 5)) = v;
}
// and back: a lane's own four columns of a block whose whole rows were written by put_patch_rows
__device__ __forceinline__ bf16x4 patch_get(char *patch, int lane, int f2, int g) {
  return *reinterpret_cast<const bf16x4 *>(patch_slot(patch, lane & 31, f2 * 4 + g) + 8 * (lane >> 5));
}
struct PatchRows {
  bf16x8 v[4];
};
__device__ __forceinline__ PatchRows read_patch_rows(char *patch, int lane) {
  PatchRows r;
#pragma unroll
  for (int it = 0; it < 4; ++it) r.v[it] = *reinterpret_cast<const bf16x8 *>(patch_slot(patch, it * 8 + (lane >> 3), lane & 7));
  return r;
}
__device__ __forceinline__ void put_patch_rows(const PatchRows &r, char *patch, int lane) {
#pragma unroll
  for (int it = 0; it < 4; ++it) *reinterpret_cast<bf16x8 *>(patch_slot(patch, it * 8 + (lane >> 3), lane & 7)) = r.v[it];
}

// Destination of one 32 x 64 block: a window and the lane's byte offset for each of its four 16-byte row chunks.
struct BlockDest {
  window_t win;
  uint32_t off[4];
  __device__ __forceinline__ void put(int it, bf16x8 v) const {
    // Non-temporal: a launch streams up to gigabytes of output through each XCD's 4 MB L2, which also holds the operand
    // panels its 32 compute units share; marking the lines for early eviction keeps them from pushing the panels out
    // (512 -> 4096, 262144 scattered rows: 1.39 -> 1.27 ms; neutral to 2 % either way on outputs of tens of MB).
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), win, (int)off[it], 0, 2);
  }
};
// The same for tensors of 4 GB and more, whose scattered rows a 32-bit offset does not reach: masked lanes store to the
// landing zone.
struct WideBlockDest {
  bf16_t *p[4];
  __device__ __forceinline__ void put(int it, bf16x8 v) const { __builtin_nontemporal_store(v, reinterpret_cast<bf16x8 *>(p[it])); }
};

template <typename Dest> struct RowStore {
  PatchRows rows;
  Dest dest;
  bool have = false;
};
template <typename Dest> __device__ __forceinline__ void issue_row_store(const RowStore<Dest> &p) {
#pragma unroll
  for (int it = 0; it < 4; ++it) p.dest.put(it, p.rows.v[it]);
}
// One block through the pipeline: write_block() fills the patch from the accumulators; the previous block's
// stores go out behind this block's LDS traffic.
template <typename Dest, typename WriteFn>
__device__ __forceinline__ void pipe_block(RowStore<Dest> &pend, char *patch, int lane, WriteFn write_block, const Dest &dest) {
  sched_fence();
  write_block();
  RowStore<Dest> cur;
  cur.rows = read_patch_rows(patch, lane);
  sched_fence();
  if (pend.have) issue_row_store(pend);
  cur.dest = dest;
  cur.have = true;
  pend = cur;
}
// accumulators of one 32 x 32 fragment pair (64 columns) -> patch, rounded to bf16
__device__ __forceinline__ void acc_block_to_patch(const f32x16 &a0, const f32x16 &a1, char *patch, int lane) {
#pragma unroll
  for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = (bf16_t)acc_read(f2 == 0 ? a0[g * 4 + q] : a1[g * 4 + q]);
      patch_put(patch, lane, f2, g, v);
    }
}

// store instructions a wavefront issues per tile, at least (a launch with fp32 partials issues more)
template <int FM, int ACT> constexpr int EpilogueStores = FM * (ACT == 1 ? 12 : ACT == 2 ? 4 : ACT == 7 ? 24 : ACT == 3 || ACT >= 5 ? 16 : 8);

// dest(fm, half): where rows fm * 32 .. + 31, columns half * 64 .. + 63 of the wavefront's tile go
template <int FM, typename DestFn>
__device__ __forceinline__ void store_wave_tile(const f32x16 (&acc)[FM][FR], char *patch, DestFn dest, int lane) {
  acc_settle();
  RowStore<decltype(dest(0, 0))> pend;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int half = 0; half < 2; ++half)
      pipe_block(pend, patch, lane, [&] { acc_block_to_patch(acc[fm][half * 2], acc[fm][half * 2 + 1], patch, lane); }, dest(fm, half));
  sched_fence();
  issue_row_store(pend);
}

// Epilogue of a SwiGLU tile: the wavefront's 128 accumulator columns are 64 gate columns (fragments 0, 1)
// and the 64 up columns that pair with them (fragments 2, 3), so a lane holds both factors of each hidden
// unit in matching registers.  Writes the pre-activation halves (KEEP) and H = silu(gate) * up, each
// through the same pipeline as above: pre(fm, 0 gate / 1 up) and hid(fm) say where.
template <bool KEEP, int FM, typename PreFn, typename HidFn>
__device__ __forceinline__ void store_wave_tile_swiglu(const f32x16 (&acc)[FM][FR], char *patch, PreFn pre, HidFn hid, int lane) {
  acc_settle();
  RowStore<BlockDest> pend;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    if (KEEP) {
#pragma unroll
      for (int half = 0; half < 2; ++half)
        pipe_block(pend, patch, lane, [&] { acc_block_to_patch(acc[fm][half * 2], acc[fm][half * 2 + 1], patch, lane); }, pre(fm, half));
    }
    pipe_block(pend, patch, lane, [&] {
#pragma unroll
      for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 v;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float gate = acc_read(acc[fm][f2][g * 4 + q]), up = acc_read(acc[fm][2 + f2][g * 4 + q]);
            float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gate));
            v[q] = (bf16_t)(gate * sig * up);
          }
          patch_put(patch, lane, f2, g, v);
        }
    }, hid(fm));
  }
  sched_fence();
  issue_row_store(pend);
}

// What the two backward epilogues read and write besides the block destinations.  The windows start at the wavefront's first row
// (expert-sorted) and end with the segment, so rows past it read zeros and are not written; `scale` is a whole array, and with PLACES
// (store_wave_tile_dp) `saved` a whole tensor, whose rows are found through `places`.
struct BwdRows {
  window_t saved;       // pre-activations [rows, 2 * n] (SwiGLU) or hidden rows [rows, n]
  const int *places;    // order indices of the wavefront's rows, always set (LDS; past the `left` rows there are, the last one's again):
                        // where their routing weights lie, and with PLACES their rows of `saved`
  int left;
  window_t scale;       // routing weight of every slot
  window_t hidden;      // hidden rows [rows, n], where they are read beside the pre-activations
  window_t dp;          // slabs of dp, [rows, part_ld] fp32
  uint32_t saved_bytes; // bytes per row of `saved`
  uint32_t part_bytes;  // bytes per row of the slabs
  uint32_t part_col;    // this wavefront's slab
  int n, gcol;          // hidden units, and the wavefront's first one
};
__device__ __forceinline__ void put_dp(const BwdRows &b, int fm, float dp, int lane) {
  dp += __shfl_xor(dp, 32, 64);
  const uint32_t off = lane < 32 ? (uint32_t)(fm * 32 + lane) * b.part_bytes + b.part_col * 4u : OFF_WINDOW;
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, dp), b.dp, (int)off, 0, 0);
}
__device__ __forceinline__ float row_weight(const BwdRows &b, int fm, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b.scale, b.places[fm * 32 + (lane & 31)] * 4, 0, 0));
}

// Epilogue of the second ParallelLinear's input-gradient product with the SwiGLU derivative and Alg. 2's dp folded in.
// The accumulators hold dH / p for 128 hidden units of 32 * FM expert-sorted rows (the product ran on the unweighted
// upstream rows).  Per 32 x 64 block the wavefront fetches the matching gate and up pre-activations (whole rows, turned to the
// accumulators' layout through the patch, the next block requested before the current one is used), forms
// h = silu(gate) * up and the partial dot <acc, h> (summed over the wavefront's 128 columns: one slab of dp), scales
// the accumulators by the row's routing weight and writes
//   dgate = dh * up * (sig + silu * (1 - sig)),  dup = dh * silu
// to the two halves of dHpre through the patch pipeline: dest(fm, half, 0 gate / 1 up).  Columns past the width read
// whatever lies there and are neither stored nor added to the dot.
struct RowWeights {
  float w[4];           // of the rows that a lane holds pieces of where eight lanes hold a row
};
__device__ __forceinline__ RowWeights row_weights(const BwdRows &b, int fm, int lane) {
  RowWeights r;
#pragma unroll
  for (int it = 0; it < 4; ++it)
    r.w[it] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b.scale, b.places[fm * 32 + it * 8 + (lane >> 3)] * 4, 0, 0));
  return r;
}
struct GateUp {
  PatchRows gt, up;
};
// A 32 x 64 block of a saved tensor as whole 128-byte rows, eight lanes each, `col` bytes into the rows.  (A lane fetching its
// own row's 8-byte pieces touched 32 lines per instruction, each line again for every piece, and more lines than the L1
// holds: the epilogue took 27 us a tile, on 54 us of products at a contraction of 2048.)
template <bool PLACES = false> __device__ __forceinline__ PatchRows load_saved_rows(const BwdRows &b, int fm, uint32_t col, int lane) {
  PatchRows r;
  if (PLACES) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int row = fm * 32 + it * 8 + (lane >> 3);
      const uint32_t off = (uint32_t)b.places[row] * b.saved_bytes + col + (uint32_t)(lane & 7) * 16u;
      r.v[it] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b.saved, (int)(row < b.left ? off : ~0u), 0, 0));
    }
    return r;
  }
  const uint32_t base = (uint32_t)(fm * 32 + (lane >> 3)) * b.saved_bytes + col + (uint32_t)(lane & 7) * 16u;
#pragma unroll
  for (int it = 0; it < 4; ++it)
    r.v[it] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b.saved, (int)(base + (uint32_t)(it * 8) * b.saved_bytes), 0, 0));
  return r;
}
__device__ __forceinline__ PatchRows load_hidden_rows(const BwdRows &b, int fm, int half, int lane) {
  PatchRows r;
  const uint32_t row = (uint32_t)b.n * 2u, base = (uint32_t)(fm * 32 + (lane >> 3)) * row + (uint32_t)(b.gcol + half * 64 + (lane & 7) * 8) * 2u;
#pragma unroll
  for (int it = 0; it < 4; ++it) r.v[it] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(b.hidden, (int)(base + (uint32_t)(it * 8) * row), 0, 0));
  return r;
}
// ... and turned to the accumulators' layout through the patch
__device__ __forceinline__ void saved_columns(const PatchRows &r, char *patch, int lane, bf16x4 (&v)[2][4]) {
  put_patch_rows(r, patch, lane);
#pragma unroll
  for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
    for (int g = 0; g < 4; ++g) v[f2][g] = patch_get(patch, lane, f2, g);
}
__device__ __forceinline__ GateUp load_gate_up(const BwdRows &b, int fm, int half, int lane) {
  const uint32_t col = (uint32_t)(b.gcol + half * 64) * 2u;
  return GateUp{load_saved_rows(b, fm, col, lane), load_saved_rows(b, fm, col + (uint32_t)b.n * 2u, lane)};
}
// HW: and Hw = p * H to dest_hw(fm, half), from the saved H: a block of it goes from whole rows to whole rows, so it needs no turn
// through the patch.  (p * h from the fp32 h at hand reads nothing more, but that h comes from gates and ups rounded to bf16: the error of
// dW2 against 64 bits was 3.45e-3 instead of 2.86e-3.)
template <bool HW, int FM, typename DestFn, typename HwFn>
__device__ __forceinline__ void store_wave_tile_swiglu_bwd(const f32x16 (&acc)[FM][FR], char *patch, const BwdRows &b, DestFn dest,
                                                           HwFn dest_hw, int lane) {
  acc_settle();
  RowStore<BlockDest> pend;
  GateUp in = load_gate_up(b, 0, 0, lane);
  float scale_next = row_weight(b, 0, lane);
  PatchRows hidden_next;
  RowWeights weights_next;
  if (HW) {
    hidden_next = load_hidden_rows(b, 0, 0, lane);
    weights_next = row_weights(b, 0, lane);
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    float dp = 0.f;
    const float scale = scale_next;
    const RowWeights weights = weights_next;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const PatchRows hidden = hidden_next;
      const GateUp rows = in;
      bf16x4 gt[2][4], up[2][4];
      sched_fence();
      saved_columns(rows.gt, patch, lane, gt);
      saved_columns(rows.up, patch, lane, up);
      sched_fence();
      if (fm * 2 + half + 1 < 2 * FM) {   // request the next 64 columns (or the next fragment row) now
        in = load_gate_up(b, half == 0 ? fm : fm + 1, half == 0 ? 1 : 0, lane);
        if (half == 1) scale_next = row_weight(b, fm + 1, lane);
        if (HW) {
          hidden_next = load_hidden_rows(b, half == 0 ? fm : fm + 1, half == 0 ? 1 : 0, lane);
          if (half == 1) weights_next = row_weights(b, fm + 1, lane);
        }
      }
      bf16x4 du[2][4];
      pipe_block(pend, patch, lane, [&] {
#pragma unroll
        for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int col = b.gcol + half * 64 + f2 * 32 + 8 * g + 4 * (lane >> 5);
            bf16x4 dg;
            float part = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float a = acc_read(acc[fm][half * 2 + f2][g * 4 + q]);
              const float gate = (float)gt[f2][g][q], u = (float)up[f2][g][q];
              const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gate));
              const float silu = gate * sig;
              part = fmaf(a, silu * u, part);
              const float dh = scale * a;
              dg[q] = (bf16_t)(dh * u * (sig + silu * (1.0f - sig)));
              du[f2][g][q] = (bf16_t)(dh * silu);
            }
            dp += col < b.n ? part : 0.f;
            patch_put(patch, lane, f2, g, dg);
          }
      }, dest(fm, half, 0));
      pipe_block(pend, patch, lane, [&] {
#pragma unroll
        for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
          for (int g = 0; g < 4; ++g) patch_put(patch, lane, f2, g, du[f2][g]);
      }, dest(fm, half, 1));
      if constexpr (HW) {
        const BlockDest to = dest_hw(fm, half);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          bf16x8 v;
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = (bf16_t)(weights.w[it] * (float)hidden.v[it][q]);
          to.put(it, v);
        }
        sched_fence();
      }
    }
    put_dp(b, fm, dp, lane);
  }
  sched_fence();
  issue_row_store(pend);
}

// The activation-agnostic form: the accumulators hold dH / p; the wavefront fetches the saved hidden activations H of the
// block, adds <acc, H> to the row's slab of dp, and writes dH = p * acc (HW: and Hw = p * H).
// PLACES: the hidden rows and dH lie in slot order, the slabs and Hw are expert-sorted.
template <bool HW, bool PLACES, int FM, typename DestFn, typename HwFn>
__device__ __forceinline__ void store_wave_tile_dp(const f32x16 (&acc)[FM][FR], char *patch, const BwdRows &b, DestFn dest,
                                                   HwFn dest_hw, int lane) {
  acc_settle();
  auto load_h = [&](int fm, int half) { return load_saved_rows<PLACES>(b, fm, (uint32_t)(b.gcol + half * 64) * 2u, lane); };
  RowStore<BlockDest> pend;
  PatchRows next = load_h(0, 0);
  float scale_next = row_weight(b, 0, lane);
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    float dp = 0.f;
    const float scale = scale_next;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const PatchRows rows = next;
      bf16x4 cur[2][4];
      sched_fence();
      saved_columns(rows, patch, lane, cur);
      sched_fence();
      if (fm * 2 + half + 1 < 2 * FM) {   // request the next 64 columns (or the next fragment row) now
        next = load_h(half == 0 ? fm : fm + 1, half == 0 ? 1 : 0);
        if (half == 1) scale_next = row_weight(b, fm + 1, lane);
      }
      pipe_block(pend, patch, lane, [&] {
#pragma unroll
        for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int col = b.gcol + half * 64 + f2 * 32 + 8 * g + 4 * (lane >> 5);
            bf16x4 v;
            float part = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float a = acc_read(acc[fm][half * 2 + f2][g * 4 + q]);
              part = fmaf(a, (float)cur[f2][g][q], part);
              v[q] = (bf16_t)(scale * a);
            }
            dp += col < b.n ? part : 0.f;
            patch_put(patch, lane, f2, g, v);
          }
      }, dest(fm, half));
      if constexpr (HW)
        pipe_block(pend, patch, lane, [&] {
#pragma unroll
          for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              bf16x4 v;
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = (bf16_t)(scale * (float)cur[f2][g][q]);
              patch_put(patch, lane, f2, g, v);
            }
        }, dest_hw(fm, half));
    }
    put_dp(b, fm, dp, lane);
  }
  sched_fence();
  issue_row_store(pend);
}

// A wavefront's accumulators as fp32 into a 256-wide partial tile (chunks of a split contraction).
template <int FM>
__device__ __forceinline__ void store_wave_partial(const f32x16 (&acc)[FM][FR], float *dst, int lane) {
  acc_settle();
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FR; ++fn) {
      sched_fence();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4 v = make_float4(acc_read(acc[fm][fn][4 * g]), acc_read(acc[fm][fn][4 * g + 1]), acc_read(acc[fm][fn][4 * g + 2]),
                               acc_read(acc[fm][fn][4 * g + 3]));
        *reinterpret_cast<float4 *>(dst + (size_t)(fm * 32 + (lane & 31)) * TB + fn * 32 + 8 * g + 4 * (lane >> 5)) = v;
      }
    }
}

}  // namespace
