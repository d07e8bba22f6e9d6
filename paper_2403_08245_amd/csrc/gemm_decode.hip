// scatter2scatter for the decoding regime (Sec. 5 names it as the open case): a few rows per
// expert, so the product is a stream of every used expert's weights past a handful of rows and
// the only thing that matters is keeping HBM busy.
//
// A block of four wavefronts owns a 32-row output tile of one expert, 128 columns per wavefront across; wavefronts that share
// columns take the contraction's 32-row steps in turn and add their sums through LDS at the end, in a fixed order.  The weights go
// from memory straight to registers: a lane loads 8 rows x 8 columns (16 bytes of each row, 256 bytes per row and sixteen
// lanes) and turns them into the operands of eight 16x16x32 matrix instructions with one byte permutation per register,
// operand j holding column j of every lane's eight.  No LDS traffic, no barrier and no swizzle in the loop, and DEPTH steps of
// 8 KB per wavefront in flight.  Weights are read once, so where a call's exceed the last-level cache they pass the caches by (64
// experts, 2048 -> 2 x 512: 53 -> 47 us; S2SArgs::call_weights says which count).
// Before, one wavefront walked a 128-column tile's whole contraction through an LDS ring: 64 tokens on 64 experts, 2048 ->
// 2 x 512 -> 2048, 57 + 29 us (4.7 TB/s); now 47 + 25 (5.7 and 5.4).  Four tokens (25 experts): 26 + 14 us; now 26 + 12.
// Forward products only (W as stored); the gradients of such small batches use the large-tile kernels.
#include "mfma_common.h"
#include <type_traits>

namespace {

constexpr int DM = 32;                        // rows of a tile: two 16-row fragments
constexpr int DN = 128;                       // columns of a wavefront
constexpr int DEPTH = 2;                      // steps in flight per wavefront (three: the same times)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct WStep {
  u32x4 row[8];      // eight contraction rows of the lane's eight columns
};
// operand j of the matrix instructions: column j of the lane, its eight contraction rows
template <int J> __device__ __forceinline__ bf16x8 w_frag(const WStep &w) {
  union { bf16x8 v; uint32_t d[4]; } u;
#pragma unroll
  for (int t = 0; t < 4; ++t) u.d[t] = __builtin_amdgcn_perm(w.row[2 * t + 1][J / 2], w.row[2 * t][J / 2], J % 2 ? 0x07060302u : 0x05040100u);
  return u.v;
}

// ACT 0: C = A W.  ACT 1 / 2: fused SwiGLU (a tile is 64 gate columns and the 64 up columns pairing with
// them), keeping / not keeping the pre-activation.
template <int ACT, bool SCATTER_OUT, int CW, int KW, bool ONCE>
__global__ void __launch_bounds__(64 * CW * KW, 2) s2s_decode_kernel(S2SArgs a, int n_chunks) {
  __shared__ float s_part[KW][CW][32][64];     // one fragment's sums of every wavefront
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int cw = wave % CW, kw = wave / CW;    // its 128 columns of the tile, its share of the contraction
  const int mt = (int)blockIdx.x / n_chunks, nc = (int)blockIdx.x - mt * n_chunks;
  int e, row0, row_end;
  if (!locate_rows<DM>(a.offsets, a.E, mt, lane, e, row0, row_end)) return;   // grid is an upper bound
  e = __builtin_amdgcn_readfirstlane(e);
  row0 = __builtin_amdgcn_readfirstlane(row0);
  row_end = __builtin_amdgcn_readfirstlane(row_end);
  const bool two = row_end - row0 > 16;              // both fragments hold rows
  const int half_n = a.N / 2;
  const int n0 = nc * CW * (ACT ? DN / 2 : DN);      // first (gate) column of the tile
  const int nh = a.K / HK;
  const int c = lane & 15, q = lane >> 4;            // the lane's column group and quarter of a step

  // First column of column group g of the wavefronts `w`.  SwiGLU: one wavefront across holds 64 gate columns and their 64 up
  // columns, several hold gates (the first half of them) or ups.
  constexpr int GATES = CW / 2;
  auto column = [&](int w, int g) {
    if (!ACT) return n0 + w * DN + g * 8;
    if (CW == 1) return n0 + (g & 7) * 8 + (g >> 3) * half_n;
    return n0 + (w % (CW > 1 ? GATES : 1)) * DN + g * 8 + (w / (CW > 1 ? GATES : 1)) * half_n;
  };
  auto exists = [&](int w, int g) {
    if (!ACT) return column(w, g) < a.N;
    const int col = column(w, g);
    return (CW == 1 ? g < 8 : w < GATES) ? col < half_n : col < a.N;
  };
  const bool have = exists(cw, c);
  const char *W = (const char *)((const bf16_t *)a.W + (size_t)e * a.w_stride);
  const uint32_t w_lane = (uint32_t)(8 * q) * (uint32_t)a.ldw * 2u + (uint32_t)(have ? column(cw, c) : 0) * 2u;
  const size_t row_bytes = (size_t)a.ldw * 2;
  // Steps kw, kw + KW, ... are this wavefront's (a share of one step requests it DEPTH times).
  auto step_at = [&](int s) { return min(kw + s * KW, nh - 1); };
  const int mine = (nh - kw + KW - 1) / KW;
  f32x4 acc[2][8];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](auto j, const WStep &ws, const bf16x8 (&xs)[2]) {
    constexpr int J = decltype(j)::value;
    const bf16x8 f = w_frag<J>(ws);
    acc[0][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, xs[0], acc[0][J], 0, 0, 0);
    if (two) acc[1][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, xs[1], acc[1][J], 0, 0, 0);
  };
  auto use = [&](const WStep &ws, const bf16x8 (&xs)[2]) {
    multiply(std::integral_constant<int, 0>{}, ws, xs);
    multiply(std::integral_constant<int, 1>{}, ws, xs);
    multiply(std::integral_constant<int, 2>{}, ws, xs);
    multiply(std::integral_constant<int, 3>{}, ws, xs);
    multiply(std::integral_constant<int, 4>{}, ws, xs);
    multiply(std::integral_constant<int, 5>{}, ws, xs);
    multiply(std::integral_constant<int, 6>{}, ws, xs);
    multiply(std::integral_constant<int, 7>{}, ws, xs);
  };
  auto contract = [&](auto past_caches) {
    auto load_w = [&](int s) {
      WStep w;
      const char *p = W + (size_t)(step_at(s) * HK) * row_bytes;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(p + (size_t)i * row_bytes + w_lane);
        w.row[i] = decltype(past_caches)::value ? __builtin_nontemporal_load(src) : *src;
      }
      return w;
    };
    WStep w[DEPTH];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) w[s] = load_w(s);

    const bf16_t *pa[2];                               // rows past the segment repeat its last row
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int i = min(row0 + m * 16 + c, row_end - 1);
      const int src = a.a_map.o ? a.a_map.o[i] / a.a_map.fan : i;
      pa[m] = (const bf16_t *)a.A + (size_t)src * a.K + q * 8;
    }
    bf16x8 x[DEPTH][2];
    auto load_x = [&](int step, bf16x8 (&v)[2]) {
      v[0] = *reinterpret_cast<const bf16x8 *>(pa[0] + step * HK);
      if (two) v[1] = *reinterpret_cast<const bf16x8 *>(pa[1] + step * HK);
    };
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) load_x(step_at(s), x[s]);
    int s = 0;
    auto refill = [&](int u) {
      w[u] = load_w(s + u + DEPTH);
      load_x(step_at(s + u + DEPTH), x[u]);
    };
    // The last steps stand by themselves: requests past the end would have every share read DEPTH * 8 KB that nothing uses, and a
    // condition on the requests in this loop would make it wait for all of them.  64 tokens on 64 experts, 2048 -> 2 x 512 ->
    // 2048: the forward pass 74.1 -> 73.2 us; 200 tokens with Zipf(1.2) loads 104 -> 100.
#pragma unroll 1
    for (; s + 2 * DEPTH <= mine; s += DEPTH) {
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        use(w[u], x[u]);
        refill(u);
      }
    }
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      if (s + u < mine) use(w[u], x[u]);
      if (s + u + DEPTH < mine) refill(u);
    }
#pragma unroll
    for (int u = 0; u < DEPTH - 1; ++u)
      if (s + u + DEPTH < mine) use(w[u], x[u]);
  };
  // An expert with more rows than one tile has its weights read again, by other blocks, which should find them in the caches (200
  // tokens on 64 experts with Zipf(1.2) loads, 2048 -> 2 x 512 -> 2048: the forward pass 116 us with all weights past the caches,
  // 107 with none, 105 so).
  if (ONCE && row_end - __builtin_amdgcn_readfirstlane(a.offsets[e]) <= DM) {
    __asm__ volatile("" ::: "memory");   // keeps the compiler from folding the two forms into one, which drops the hint
    contract(std::true_type{});
  } else {
    contract(std::false_type{});
  }

  // Sums over the contraction's shares, in their order.  Lane (c, q) holds row c of the fragment and, in element r of the
  // accumulators, columns 0..7 (j) of column group 4 * q + r.
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    if (m == 1 && !two) break;
    if (m == 1) __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_part[kw][cw][r * 8 + j][lane] = acc[m][j][r];
    __syncthreads();
    const int i = row0 + m * 16 + c;
    auto rounded = [](const float (&v)[8]) {
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (bf16_t)v[j];
      return o;
    };
    constexpr int ACROSS = ACT && CW > 1 ? GATES : CW;
    for (int t = wave; t < ACROSS * 4; t += CW * KW) {   // element r of every lane of the wavefronts w
      const int w = t / 4, r = t % 4, g = 4 * q + r;
      auto total = [&](int from, int from_lane, float (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          v[j] = 0.f;
#pragma unroll
          for (int p = 0; p < KW; ++p) v[j] += s_part[p][from][r * 8 + j][from_lane];
        }
      };
      if (ACT == 0) {
        float v[8];
        total(w, lane, v);
        if (i < row_end && exists(w, g)) {
          const size_t dst = SCATTER_OUT ? (size_t)a.c_map.o[i] : (size_t)i;
          *reinterpret_cast<bf16x8 *>((bf16_t *)a.C + dst * a.N + column(w, g)) = rounded(v);
        }
      } else if (CW > 1 || q < 2) {   // one wavefront across: column groups 0..7 are gates, 8..15 (lane + 32) their ups
        float gate[8], up[8], h[8];
        total(w, lane, gate);
        if (CW > 1) total(w + GATES, lane, up);
        else total(w, lane + 32, up);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gate[j]));
          h[j] = gate[j] * sig * up[j];
        }
        const int col = column(w, g);
        if (i < row_end && col < half_n) {
          if (ACT == 1) {
            bf16_t *Hpre = (bf16_t *)a.C + (size_t)i * a.N;
            *reinterpret_cast<bf16x8 *>(Hpre + col) = rounded(gate);
            *reinterpret_cast<bf16x8 *>(Hpre + half_n + col) = rounded(up);
          }
          *reinterpret_cast<bf16x8 *>((bf16_t *)a.H + (size_t)i * half_n + col) = rounded(h);
        }
      }
    }
  }
}

template <int ACT, bool SCATTER_OUT, int CW, int KW> int launch_decode_as(hipStream_t s, const S2SArgs &a) {
  const int n_chunks = ACT ? ceil_div(a.N / 2, CW * DN / 2) : ceil_div(a.N, CW * DN);
  const long long m_bound = a.Tk / DM + a.E;           // >= sum_e ceil(n_e / 32)
  const dim3 grid((unsigned)(m_bound * n_chunks)), block(64 * CW * KW);
  if (weights_pass_caches(a)) hipLaunchKernelGGL((s2s_decode_kernel<ACT, SCATTER_OUT, CW, KW, true>), grid, block, 0, s, a, n_chunks);
  else hipLaunchKernelGGL((s2s_decode_kernel<ACT, SCATTER_OUT, CW, KW, false>), grid, block, 0, s, a, n_chunks);
  SMOE_LAUNCH_CHECK();
  return SMOE_OK;
}
// Four wavefronts: as many of them side by side as leave a tile for every compute unit, the rest share the contraction.  Wide
// tiles read longer runs of a row of W (64 experts, weights not in the cache: 2048 -> 2 x 512 in 55 us one across, 47 two
// across, 56 four across on half the chip; 512 -> 2048 in 29, 27, 25 us), narrow ones fill the chip (25 experts: 2048 -> 2 x 512
// in 26 us one across, 31 two).
template <int ACT, bool SCATTER_OUT> int launch_decode(hipStream_t s, const S2SArgs &a) {
  const long long experts = a.Tk < a.E ? a.Tk : a.E;
  auto tiles = [&](int cw) { return experts * ceil_div(ACT ? a.N / 2 : a.N, ACT ? cw * DN / 2 : cw * DN); };
  if (tiles(4) >= a.grid) return launch_decode_as<ACT, SCATTER_OUT, 4, 1>(s, a);
  if (tiles(2) >= a.grid) return launch_decode_as<ACT, SCATTER_OUT, 2, 2>(s, a);
  return launch_decode_as<ACT, SCATTER_OUT, 1, 4>(s, a);
}

}  // namespace

// The decoding regime: on average at most one 32-row tile per expert.  Gathered or expert-sorted input,
// W as stored, any output order; widths as the 16-byte loads and stores need them, and rows of W that 24 of them fit a
// lane's 32-bit offset.
// The line at 32 rows per expert, forward pass of the layer in us, these kernels / the large tiles (uniform router, other tokens
// at every call):
//   8 experts, 1024 -> 2 x 2816 -> 1024: 8 rows 35 / 57, 24 rows 39 / 58, 32 rows 46 / 59, 64 rows 55 / 60, 96 rows 58 / 62;
//   32 experts, 1024 -> 512 -> 1024: 8 rows 23 / 41, 32 rows 29 / 42, 64 rows 38 / 43, 96 rows 41 / 45;
//   8 experts, 4096 -> 2 x 14336 -> 4096: 8 rows 434 / 581, 24 rows 476 / 594, 32 rows 644 / 597;
//   16 experts, 4096 -> 2 x 1024 -> 4096: 8 rows 80 / 104, 20 rows 87 / 105, 24 rows 105 / 106, 32 rows 115 / 107;
//   64 experts, 2048 -> 512 -> 2048: 8 rows 53 / 70, 20 rows 62 / 74, 24 rows 80 / 75, 32 rows 87 / 77;
//   64 experts, 2048 -> 2 x 512 -> 2048: 8 rows 73 / 78, 18 rows 78 / 82, 22 rows 100 / 82, 32 rows 120 / 85;
//   128 experts, the same: 8 rows 133 / 152, 18 rows 143 / 157, 22 rows 190 / 159, 32 rows 217 / 162.
// So it is late for layers whose weights exceed the last-level cache and whose tiles are about one per compute unit: as soon as
// one expert has more than 32 rows, some compute units get a second tile and the launch lasts longer by half.  A line drawn from
// the number of experts expected above 32 rows and the tiles per compute unit won 1.3 to 1.6 times there, but lost where tiles are
// fewer (24 experts, 3072 -> 1024 -> 3072, 25 rows: 84 -> 111) or contractions long (8 experts, 14336, 25 rows: 518 -> 588); where it
// lies under uneven routing depends on counts that only the device has.  So it stays at a tile for the average expert.
bool s2s_decode_supported(const S2SArgs &a) {
  if (a.trans_w || a.Tk <= 0 || a.E < 1 || (long long)a.Tk > (long long)DM * a.E) return false;
  if (a.K < HK || a.K % HK || a.N % 8 || a.ldw % 8 || a.ldw > (1 << 25)) return false;
  if (a.H && (a.N % 16 || a.c_map.o)) return false;
  const long long blocks = ((long long)a.Tk / DM + a.E) * ceil_div(a.N, DN / 2);
  return blocks * 256 <= 0xffffffffLL;
}

int launch_s2s_decode(hipStream_t s, const S2SArgs &a) {
  if (!s2s_decode_supported(a)) return SMOE_ERR_UNSUPPORTED;
  if (a.H) return a.C ? launch_decode<1, false>(s, a) : launch_decode<2, false>(s, a);
  return a.c_map.o ? launch_decode<0, true>(s, a) : launch_decode<0, false>(s, a);
}
