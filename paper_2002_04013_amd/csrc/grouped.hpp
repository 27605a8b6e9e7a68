// Launch helpers shared by the expert blocks: the device-side tile plan of a grouped
// GEMM, per-expert column sums, and the tile shapes and launches of the two grouped
// GEMM implementations (gemm_f32.hpp: fp32; gemm2.hpp: bf16).
#pragma once
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <utility>

#include "common.hpp"
#include "gemm.hpp"
#include "gemm2.hpp"
#include "gemm_f32.hpp"

namespace dmoe {

// Tile plans of one FFN call, from the expert row offsets:
//   plan_a[e], plan_b[e] = sum over experts before e of ceil(rows / BM) for two tile heights
//                          (GROUP_M m-tiles; the GEMMs of a call use at most two)
//   act[e]               = number of experts before e that have rows (GROUP_K experts)
// with the totals at [N]; act may be null.  A GEMM with NT n-tiles (GROUP_M) or MT*NT tiles
// per expert (GROUP_K) scales these.  One block: wave w owns the experts [64 G w, 64 G (w + 1)),
// 64 at a time, so that loads and stores are whole lines; a shuffle scan of every 64, the waves'
// sums meet in LDS once.  Tile heights are multiples of 32, and a division by the multiple is a
// multiplication.  (A thread owning G consecutive experts had strided accesses: 15625 experts
// 29 us for one height, 31 for two, 39 with act; 15 now with all, and 3.9 where it was 4.8 for 64 experts.)
constexpr int TP_WAVES = 16;
struct TileHeight {
  int mul; uint32_t inv;                           // in 32-row blocks, and 2^32 / mul rounded up
  __device__ __forceinline__ int tiles(int rows) const {
    // exact below 2^28 blocks: the error of inv is at most mul / 2^32 a block, mul <= 9
    const uint32_t n = (uint32_t)((rows + 31) >> 5) + (uint32_t)(mul - 1);
    return mul == 1 ? (int)n : (int)__umulhi(n, inv);
  }
};
static TileHeight tile_height(int BM) {
  const uint32_t mul = (uint32_t)(BM / 32);
  return {(int)mul, mul > 1 ? (uint32_t)(((1ull << 32) + mul - 1) / mul) : 0u};
}
static __global__ void __launch_bounds__(64 * TP_WAVES)
tile_plan(const int32_t* offsets, int N, TileHeight ha, TileHeight hb, int32_t* plan_a, int32_t* plan_b, int32_t* act) {
  __shared__ int part[3][TP_WAVES];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = (N + 64 * TP_WAVES - 1) / (64 * TP_WAVES), base = 64 * G * wave;
  struct Group { int ta, tb, ia, ib; uint64_t has; };   // this lane's tiles, and inclusive sums over the lanes
  auto rows = [&](int e) { return e < N ? offsets[e + 1] - offsets[e] : 0; };
  auto scan = [&](int c) {
    Group g;
    g.ta = g.ia = ha.tiles(c);
    g.tb = g.ib = hb.tiles(c);
    g.has = __ballot(c > 0);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int va = __shfl_up(g.ia, o, 64), vb = __shfl_up(g.ib, o, 64);
      if (lane >= o) { g.ia += va; g.ib += vb; }
    }
    return g;
  };
  Group first = scan(rows(base + lane));
  int sa = 0, sb = 0, sn = 0;
#pragma unroll 4
  for (int i = 1; i < G; ++i) {
    const int c = rows(base + 64 * i + lane);
    sa += ha.tiles(c);
    sb += hb.tiles(c);
    sn += __popcll(__ballot(c > 0));
  }
  if (G > 1) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { sa += __shfl_xor(sa, o, 64); sb += __shfl_xor(sb, o, 64); }
  }
  if (lane == 63) {
    part[0][wave] = first.ia + sa;
    part[1][wave] = first.ib + sb;
    part[2][wave] = __popcll(first.has) + sn;
  }
  __syncthreads();
  int run[3] = {0, 0, 0}, total[3] = {0, 0, 0};
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int w = 0; w < TP_WAVES; ++w) {
      const int v = part[i][w];
      run[i] += w < wave ? v : 0;
      total[i] += v;
    }
  for (int i = 0; i < G; ++i) {
    const int e = base + 64 * i + lane;
    const Group g = i == 0 ? first : scan(rows(e));
    if (e < N) {
      plan_a[e] = run[0] + g.ia - g.ta;
      plan_b[e] = run[1] + g.ib - g.tb;
      if (act) act[e] = run[2] + __popcll(g.has & ((1ull << lane) - 1ull));
    }
    run[0] += __builtin_amdgcn_readlane(g.ia, 63);
    run[1] += __builtin_amdgcn_readlane(g.ib, 63);
    run[2] += __popcll(g.has);
  }
  if (threadIdx.x == 0) {
    plan_a[N] = total[0];
    plan_b[N] = total[1];
    if (act) act[N] = total[2];
  }
}

// The plans in a call's scratch: tile heights for outputs of H (a) and D (b) columns.
struct Plan { int32_t *a, *b, *act; };
static Plan plan_at(int32_t* mem, int64_t N, bool with_act) {
  return {mem, mem + N + 1, with_act ? mem + 2 * (N + 1) : nullptr};
}
static void run_tile_plan(const Shape& s, const int32_t* offsets, int BMa, int BMb, const Plan& pl, hipStream_t st) {
  DMOE_LAUNCH(tile_plan, dim3(1), dim3(64 * TP_WAVES), 0, st, offsets, (int)s.N, tile_height(BMa), tile_height(BMb), pl.a, pl.b,
              pl.act);
}

// Column sums over each expert's rows, for the bias gradients (and the LayerNorm scale and
// shift gradients of ffblock.hip).  Bound by the one read of X.  A block takes CL * VEC columns
// of one expert and splits its rows over CS_NT / CL slices: slice s adds the rows s, s + slices,
// ... in order, the slices meet in LDS in slice order.
//   * 16 lanes, 16 slices for many rows: whole rows to a thread left a layer of few experts with
//     a few dozen blocks (64 experts of 2048 rows, 1024 bf16 columns, 268 MB 537 -> 44 us, 6.1
//     TB/s; 25 experts of 324 rows, 3008 and 960 columns in one launch 154 -> 13 us).
//   * With few rows most slices have none and the blocks are too many.  Column sums / LayerNorm
//     parameter sums in us, 256 / 64 / 16 lanes: 1024 experts, 512 and 2048 columns, 48 rows
//     50 + 86 / 41 + 81 / 39 + 86; 16 rows 19 + 37 / 18 + 36 / 23 + 50; 8 rows 12 + 24 /
//     12 + 25 / 20 + 43; 15625 experts, 8 rows 133 + 228 / 120 + 219 / 237 + 486; 2 rows 40 + 76 /
//     49 + 116 / 186 + 406; a row to 50 experts 17 + 17 / 37 + 36 / 73 + 71; 128 and 512 columns,
//     2 rows 29 + 45 / 23 + 37 / 53 + 114.  Few blocks of 64 lanes leave units idle: LayerNorm
//     backward of 16 experts of 32 rows, 2048 columns, 16 us with 64 lanes, 12 with 16.
constexpr int CS_NT = 256;
template <typename E>
static int colsum_lanes(const Shape& s, int ncols) {
  if (s.P < s.N || (s.P < 4 * s.N && ncols >= CS_NT / 2 * (16 / (int)sizeof(E)))) return 256;
  const int64_t blocks = s.N * ((ncols + 64 * (16 / (int)sizeof(E)) - 1) / (64 * (16 / (int)sizeof(E))));
  return s.P < 16 * s.N || (s.P < 48 * s.N && blocks >= 1536) ? 64 : 16;
}
// f(lanes as a compile-time constant)
template <typename F> static void with_lanes(int CL, F&& f) {
  if (CL == 256) f(std::integral_constant<int, 256>{});
  else if (CL == 64) f(std::integral_constant<int, 64>{});
  else f(std::integral_constant<int, 16>{});
}

struct ColsumJob { const void* X; void* out; int ncols, blocks; };   // X rows are ncols apart

template <typename E>
static int colsum_blocks(int ncols, int CL) {
  const int W = CL * (16 / (int)sizeof(E));
  return (ncols + W - 1) / W;
}

// acc[NS][VEC] of this thread summed over the block's slices, left in the threads of slice 0
template <int CL, int NS, int VEC>
__device__ __forceinline__ void colsum_slices(float (&acc)[NS][VEC]) {
  constexpr int SL = CS_NT / CL;
  if constexpr (SL > 1) {
    __shared__ float red[SL - 1][NS][VEC][CL];
    const int l = threadIdx.x % CL, sl = threadIdx.x / CL;
    if (sl > 0) {
#pragma unroll
      for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int i = 0; i < VEC; ++i) red[sl - 1][n][i][l] = acc[n][i];
    }
    __syncthreads();
    if (sl == 0) {
      for (int q = 0; q < SL - 1; ++q)
#pragma unroll
        for (int n = 0; n < NS; ++n)
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[n][i] += red[q][n][i][l];
    }
  }
}

// out[e][c] = sum of rows [offsets[e], offsets[e+1]) of column c (experts without rows
// are left untouched); SGD: out[e][c] -= lr * that sum (out holds the parameters).
// Two matrices in one launch: blocks [0, j0.blocks) of x sum j0, the rest j1.
template <typename E, bool SGD, int CL>
__global__ void __launch_bounds__(CS_NT)
segment_colsum(ColsumJob j0, ColsumJob j1, const int32_t* offsets, float lr) {
  constexpr int VEC = 16 / sizeof(E), S = CS_NT / CL;
  const int e = blockIdx.y;
  const int r0 = offsets[e], r1 = offsets[e + 1];
  if (r1 == r0) return;
  const bool second = (int)blockIdx.x >= j0.blocks;
  const ColsumJob& j = second ? j1 : j0;
  const int c = (((int)blockIdx.x - (second ? j0.blocks : 0)) * CL + (int)threadIdx.x % CL) * VEC;
  const bool cok = c < j.ncols;
  const E* X = reinterpret_cast<const E*>(j.X) + (cok ? c : 0);
  const int64_t ld = j.ncols;
  float acc[1][VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[0][i] = 0.f;
  // four loads in flight at a time
  constexpr int U = 4;
  // Lanes past the last column only meet the others.  One slice: r is the same in every lane, and
  // known to be (an expert of 200 rows among 1000 experts, LayerNorm parameter sums with ReLU, fp32:
  // 29 us so, 61 with a row of its own for each lane).
  if (S == 1 && !cok) return;
  int r = S == 1 ? r0 : cok ? r0 + (int)threadIdx.x / CL : r1;
  for (; r + (U - 1) * S < r1; r += U * S) {
    uint4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = *reinterpret_cast<const uint4*>(X + (int64_t)(r + u * S) * ld);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v[VEC];
      Vec<E>::unpack(q[u], v);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[0][i] += v[i];
    }
  }
  for (; r < r1; r += S) {
    float v[VEC];
    Vec<E>::unpack(*reinterpret_cast<const uint4*>(X + (int64_t)r * ld), v);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[0][i] += v[i];
  }
  colsum_slices<CL>(acc);
  if ((int)threadIdx.x >= CL || !cok) return;
  uint4* op = reinterpret_cast<uint4*>(reinterpret_cast<E*>(j.out) + (int64_t)e * j.ncols + c);
  if constexpr (SGD) {
    float w[VEC];
    Vec<E>::unpack(*op, w);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[0][i] = w[i] - lr * acc[0][i];
  }
  *op = Vec<E>::pack(acc[0]);
}

// out0[e] = column sums of X0 [rows, n0]; with X1, out1[e] = those of X1 [rows, n1]
template <typename E, bool SGD = false>
static void run_colsum(const Shape& s, const int32_t* offsets, const E* X0, int n0, E* out0, const E* X1, int n1,
                       E* out1, float lr, hipStream_t st) {
  with_lanes(colsum_lanes<E>(s, std::max(n0, n1)), [&](auto CLc) {
    constexpr int CL = decltype(CLc)::value;
    const ColsumJob j0{X0, out0, n0, colsum_blocks<E>(n0, CL)};
    const ColsumJob j1{X1, out1, n1, X1 ? colsum_blocks<E>(n1, CL) : 0};
    DMOE_LAUNCH_NAMED("segment_colsum", (segment_colsum<E, SGD, CL>), dim3((unsigned)(j0.blocks + j1.blocks), (unsigned)s.N),
                      dim3(CS_NT), 0, st, j0, j1, offsets, lr);
  });
}

constexpr int MAX_DEVICES = 64;

// The current device, or -1 when it cannot be told or is beyond MAX_DEVICES.
static int current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return -1;
  return dev;
}

// Process state of the library: per device, the compute-unit count and each GEMM
// kernel's resident blocks per compute unit, queried on first use.  Slots are atomics
// (0 = not yet known); threads that race on a first query store the same value.
static int device_cus() {
  static std::atomic<int> cus[MAX_DEVICES];
  const int dev = current_device();
  if (dev < 0) return 256;
  int c = cus[dev].load(std::memory_order_relaxed);
  if (!c) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) v = 0;
    c = v > 0 ? v : 256;
    cus[dev].store(c, std::memory_order_relaxed);
  }
  return c;
}

// Resident blocks per compute unit of kernel `kern` with `nt` threads and `lds` bytes
// of dynamic LDS, cached in `slot` (one per kernel instantiation and device); opts the
// kernel into dynamic LDS beyond 64 KiB first.
static int blocks_per_cu(std::atomic<int>* slots, const void* kern, int nt, size_t lds) {
  const int dev = current_device();
  int nb = dev >= 0 ? slots[dev].load(std::memory_order_relaxed) : 0;
  if (!nb) {
    if (lds > 65536) (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, nt, lds) != hipSuccess || nb < 1) nb = 1;
    (void)hipGetLastError();
    if (dev >= 0) slots[dev].store(nb, std::memory_order_relaxed);
  }
  return nb;
}

// fp32 path (gemm_f32.hpp); C: the tile shape
template <int GM, bool AT, bool BT, int EPI, typename C>
static void run_gemm_f32(GemmArgs<float> p, int64_t tiles_ub, hipStream_t st) {
  if (tiles_ub <= 0) return;
  auto kern = grouped_gemm_f32<GM, AT, BT, EPI, C::BM, C::BN, C::WM, C::WN, C::ST>;
  constexpr int NT = 64 * C::WM * C::WN;
  const size_t lds = gemm_f32_lds_bytes<C::BM, C::BN, C::ST>();
  static std::atomic<int> per_cu[MAX_DEVICES];
  static const char* name = [] {
    static char b[96];
    snprintf(b, sizeof b, "grouped_gemm_f32<GM=%d,AT=%d,BT=%d,EPI=%d,%dx%d>", GM, (int)AT, (int)BT, EPI, C::BM, C::BN);
    return b;
  }();
  const int nb = blocks_per_cu(per_cu, (const void*)kern, NT, lds);
  const int64_t resident = (int64_t)nb * device_cus();
  const int grid = (int)std::min<int64_t>(tiles_ub, resident);
  p.chunked = grid >= 8;
  DMOE_LAUNCH_NAMED(name, kern, dim3(grid), dim3(NT), lds, st, p);
}

// gfx950 bf16 path: direct-to-LDS multi-stage GEMM (gemm2.hpp)
template <int GM, bool AT, bool BT, int EPI, int BM, int BN, int WM, int WN, int ST, int BK, int STO = STORE_DIRECT,
          int XB = 0>
static void run_gemm2(GemmArgs<bf16> p, int64_t tiles_ub, hipStream_t st) {
  if (tiles_ub <= 0) return;
  auto kern = grouped_gemm2<GM, AT, BT, EPI, BM, BN, WM, WN, ST, 1, BK, STO, XB>;
  constexpr int NT = 64 * WM * WN;
  const size_t lds = gemm2_lds_bytes<BM, BN, ST, AT, BT, BK, WM * WN, STO, XB>();
  static std::atomic<int> per_cu[MAX_DEVICES];
  static const char* name = [] {
    static char b[96];
    snprintf(b, sizeof b, "grouped_gemm2<GM=%d,AT=%d,BT=%d,EPI=%d,%dx%d,ST=%d,BK=%d%s>", GM, (int)AT, (int)BT, EPI,
             BM + 32 * XB, BN, ST, BK, XB ? ",XB" : "");
    return b;
  }();
  const int nb = blocks_per_cu(per_cu, (const void*)kern, NT, lds);
  const int64_t resident = (int64_t)nb * device_cus();
  const int grid = (int)std::min<int64_t>(tiles_ub, resident);
  p.chunked = grid >= 8;
  DMOE_LAUNCH_NAMED(name, kern, dim3(grid), dim3(NT), lds, st, p);
}

template <typename E>
static GemmArgs<E> args_m(const int32_t* offsets, const int32_t* tpre, int scale, int N) {
  GemmArgs<E> p{};
  p.offsets = offsets; p.tprefix = tpre; p.tscale = scale; p.groups = N;
  return p;
}

// fp32 tile shapes.  64 x 64 tiles of four waves, 48 KB of ring: three blocks share a
// compute unit.  Measured at 16 experts of about 256 rows, D = 512, H = 2048 (8.6 GFLOP a
// launch): 101 (up), 109 (down), 101 (dh), 110 (dx) and 93 us (weight gradients); two
// stages (five blocks a unit) 101 to 109 us, 128 x 64 tiles 107, 131, 109, 137 and 88 us
// (fewer tiles than units for the narrow outputs), two waves 128 to 186 us.  With few rows
// per expert 32 x 64 tiles of two waves, one stage deeper (weight streaming).  Weight
// gradients of many rows: 64 x 128 tiles of eight waves, 89 us against 96 in the same run.
struct CfgF32       { static constexpr int BM = 64, BN = 64, WM = 2, WN = 2, ST = 3, TMR = BM; };
struct CfgF32DW     { static constexpr int BM = 64, BN = 128, WM = 2, WN = 4, ST = 2; };
struct CfgF32Skinny { static constexpr int BM = 32, BN = 64, WM = 1, WN = 2, ST = 4, TMR = BM; };

// bf16 tile shapes of the gemm2 path: many rows per expert -> 256x256 tiles, 8 waves,
// 64-deep k, 2 stages (best of the measured shapes at the wide workload for all three
// operand layouts); few rows -> 32x256 tiles, 4 waves, 4 stages (weight streaming).
// Weight gradients contract over an expert's rows: 64-deep k-steps when experts hold
// many rows, 32-deep ones when they hold few (a k-step past an expert's last row is
// zero-filled in LDS and still multiplied, so with ~16 rows per expert a 64-deep step
// spends three quarters of its MFMA and LDS reads on zeros).
// Weight-gradient tiles write their 128 KiB of output through LDS as whole 128-byte
// lines with the non-temporal hint: the 64 GiB of weight gradients per step then
// stream past the L2 instead of evicting the GEMM's operands from it.
// Many rows per expert: the 256-row tiles take a ninth, shared 32-row block (XB), so an
// m-tile holds up to 288 rows and an expert's rows split evenly over its m-tiles (an
// expert of 512 + 18 rows gets two tiles of 9 and 8 blocks instead of a third tile of
// one block that streams the expert's weights once more).
struct G2Fat     { static constexpr int BM = 256, BN = 256, WM = 4, WN = 2, ST = 2, BK = 64, XB = 1,
                   TMR = BM + 32 * XB; };
struct G2Skinny  { static constexpr int BM = 32, BN = 256, WM = 1, WN = 4, ST = 4, BK = 64, XB = 0, TMR = BM; };
// Between the two, and for few weights:
// G2Narrow: half the columns of G2Skinny, two blocks to a compute unit: twice the tiles.
// G2Mid64, G2Mid: 64 or 128 rows by 128 columns, two blocks to a unit.
struct G2Narrow  { static constexpr int BM = 32, BN = 128, WM = 1, WN = 4, ST = 4, BK = 64, XB = 0, TMR = BM; };
struct G2Mid64   { static constexpr int BM = 64, BN = 128, WM = 2, WN = 2, ST = 3, BK = 64, XB = 0, TMR = BM; };
struct G2Mid     { static constexpr int BM = 128, BN = 128, WM = 4, WN = 2, ST = 2, BK = 64, XB = 0, TMR = BM; };
struct G2DW      { static constexpr int BM = 256, BN = 256, WM = 4, WN = 2, ST = 2, BK = 64,
                   STO = STORE_STAGED_NT; };
struct G2DWShort { static constexpr int BM = 256, BN = 256, WM = 4, WN = 2, ST = 4, BK = 32,
                   STO = STORE_STAGED_NT; };

// weight gradients: 64-deep k-steps from an average of 96 rows per expert on
static bool deep_wgrad(const Shape& s) { return s.P >= (int64_t)96 * s.N; }

// The row-grouped tile shape for an output of n columns: row_tile_line's; from 24 rows per
// expert on the lowest estimate's, below, where the line's is 10% above it, and the outer shape
// for the rows (G2Skinny below 96 per expert, else G2Fat) where its estimate is no higher.
//
// A shape's time is its rounds over the units, R (a + K/64 (b + c rho)) with rho the 32-row
// blocks a tile holds, and what it streams, w / u + (v - w) / v0 with w the weights of the
// experts with rows and v the weights every m-tile streams (MB), the larger of the two with a
// soft corner, plus a start.  m-tiles of an expert: rows spread by sqrt(r) and 5%, as routing
// by a fresh gate spreads them.  The coefficients (us) are a least-squares fit to the
// launches of 1196 layers: 2 to 1024 experts, 4 to 4096 rows each, five (d_model, hidden) from
// 256 x 4096 to 2048 x 2048; up, down and their data gradients, each in every shape.  Over those
// 4784 launches the choice is 2% above the best shape and 20% below the outer shapes alone
// (geometric means), and more than 3% above the latter in 119; the line rule alone was 6.6%
// above the best and slower than the outer shapes in 459, most where experts fill one or two
// G2Fat tiles.  Measured in us, G2Skinny / G2Narrow / G2Mid64 / G2Mid / G2Fat:
//   256 experts, n = 1024, K = 4096, r = 160: 916 / 969 / 679 / 804 / 489
//   1024 experts, n = 2048, K = 2048, r = 80: 2230 / 2571 / 3154 / 2010 / 1982
//   16 experts, n = 1024, K = 4096, r = 80: 47 / 49 / 42 / 61 / 81; r = 1024: 368 / 356 / 243 /
//   206 / 143
//   2 experts, n = 1024, K = 512, r = 512: 15 / 12 / 14 / 14 / 33
enum RowTile { RT_SKINNY, RT_NARROW, RT_MID64, RT_MID, RT_FAT };
struct RowCost { int rows, cols, per_cu; double a, b, c, u, v0, start; };
constexpr RowCost ROW_COST[5] = {
    {G2Skinny::TMR, G2Skinny::BN, 1, 5.14, 0.372, 0.130, 5.47, 20.1, 4.57},
    {G2Narrow::TMR, G2Narrow::BN, 2, 3.99, 0.279, 0.068, 5.37, 15.3, 3.55},
    {G2Mid64::TMR, G2Mid64::BN, 2, 6.65, 0.383, 0.074, 5.11, 11.0, 2.84},
    {G2Mid::TMR, G2Mid::BN, 2, 9.85, 0.380, 0.063, 4.64, 5.98, 0.16},
    {G2Fat::TMR, G2Fat::BN, 1, 13.7, 0.495, 0.138, 4.45, 3.25, 1.76},
};
static double row_cost(const RowCost& q, double act, double r, double n, double K, double cus) {
  double mt = r / q.rows + 0.5;                              // m-tiles of an expert with rows
  if (r < 8.0 * q.rows) {
    const double sd = std::sqrt(r + 0.0025 * r * r);
    mt = 1.0;
    for (double at = q.rows; at < r + 2.0 * sd; at += q.rows)
      mt += std::min(1.0, std::max(0.0, 0.5 + (r - at) / (4.0 * sd)));
  }
  const double tiles = act * mt * std::ceil(n / q.cols);
  const double rounds = std::max(1.0, std::ceil(tiles / (cus * q.per_cu) - 0.06));
  const double w = act * n * K * 2e-6;
  const double x = rounds * (q.a + K / 64.0 * (q.b + q.c * r / mt / 32.0));
  const double y = w / q.u + w * (mt - 1.0) / q.v0;
  return std::sqrt(std::sqrt(x * x * x * x + y * y * y * y)) + q.start;
}
// By lines on the rows per expert, the weights touched and the tile counts:
//   * r < 24 (weight streaming): G2Skinny; G2Narrow when the weights that can be touched are
//     under 512 MiB, where a call is a few tiles per unit and their latency counts (up and down
//     projection in us: 4 experts of 1024 x 4096 touched 18.7 + 39.0 -> 14.8 + 29.5, 55 experts
//     94.9 + 112.1 -> 84.4 + 91.5, but 256 experts 241 -> 256, down).
//   * G2Mid, or G2Fat where its rounds over the units cost less: a round of G2Fat tiles (one
//     block to a unit) takes about 1.65 rounds of G2Mid tiles (two to a unit).
//   * fewer G2Mid tiles than compute units (narrow outputs of few experts): G2Narrow below 48
//     rows, else G2Mid64 (down projection of 16 experts in us, in the order above: 32 rows
//     45 / 31 / 40 / 54 / 73; 64 rows 46 / 45 / 43 / 56 / 77; 150 rows 92 / 70 / 60 / 64 / 93).
static RowTile row_tile_line(double act, double r, double n, double K, double cus) {
  if (r < 24.0) return act * n * K * 2.0 < 536870912.0 ? RT_NARROW : RT_SKINNY;
  auto rounds = [&](const RowCost& q) {
    const double t = act * std::max(1.0, r / q.rows + 0.5) * std::ceil(n / q.cols);
    return std::pair<double, double>(t, std::ceil(t / (cus * q.per_cu)));
  };
  const auto mid = rounds(ROW_COST[RT_MID]);
  if (mid.first < cus) return r < 48.0 ? RT_NARROW : RT_MID64;
  return 1.65 * rounds(ROW_COST[RT_FAT]).second <= mid.second ? RT_FAT : RT_MID;
}
// A plan's tile height is shared by every GEMM of an output width, so from 24 rows on the
// choice takes the other of D and H for K; below, both shapes are 32 rows high.
static RowTile row_tile(const Shape& s, int64_t n, int64_t K_gemm) {
  const double act = (double)std::min<int64_t>(s.N, s.P), r = (double)s.P / act, cus = (double)device_cus();
  if (s.P < 24 * s.N) return row_tile_line(act, (double)s.P / (double)s.N, (double)n, (double)K_gemm, cus);
  const double K = (double)(n == s.H ? s.D : s.H);
  int pick = row_tile_line(act, (double)s.P / (double)s.N, (double)n, K, cus);
  double t[5];
  for (int i = 0; i < 5; ++i) t[i] = row_cost(ROW_COST[i], act, r, (double)n, K, cus);
  const int best = (int)(std::min_element(t, t + 5) - t);
  const int outer = s.P >= 96 * s.N ? RT_FAT : RT_SKINNY;
  if (t[pick] > 1.1 * t[best]) pick = best;
  return (RowTile)(t[outer] <= t[pick] ? outer : pick);
}
static int row_tile_rows(const Shape& s, int64_t n) { return ROW_COST[row_tile(s, n, 1)].rows; }

// One row-grouped GEMM in the tile shape row_tile picks: p.tscale and the grid are set here.
template <bool BT, int EPI>
static void run_gemm2_rows(const Shape& s, GemmArgs<bf16> p, hipStream_t st) {
  auto go = [&](auto cfg) {
    using C = decltype(cfg);
    const int nt = (p.N + C::BN - 1) / C::BN;
    const int64_t mt_ub = (s.P + C::TMR - 1) / C::TMR + std::min<int64_t>(s.N, s.P);
    p.tscale = nt;
    run_gemm2<GROUP_M, false, BT, EPI, C::BM, C::BN, C::WM, C::WN, C::ST, C::BK, STORE_DIRECT, C::XB>(p, mt_ub * nt, st);
  };
  switch (row_tile(s, p.N, p.K)) {
    case RT_SKINNY: go(G2Skinny{}); break;
    case RT_NARROW: go(G2Narrow{}); break;
    case RT_MID64: go(G2Mid64{}); break;
    case RT_MID: go(G2Mid{}); break;
    case RT_FAT: go(G2Fat{}); break;
  }
}

// fp32: 64-row tiles from an average of 48 rows per expert on
static bool use_fat_f32(const Shape& s) { return s.P >= (int64_t)48 * s.N; }

}  // namespace dmoe
