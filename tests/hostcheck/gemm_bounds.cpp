// Host address check of the grouped GEMMs (gemm2.hpp, gemm_f32.hpp): every thread of every block
// of each launch the layer makes runs the kernel source on the CPU, one thread after another.
// The matrix and cross-lane operations produce data only, which steers no address; global
// buffers and the LDS are allocated at their exact sizes under AddressSanitizer, so an
// access outside them stops the run with its stack.  The launches are set up as the
// layer's forward, backward, fused-SGD and LayerNorm-block entry points set them up, on
// ragged routings (an empty expert, a heavy one, row counts around tile boundaries), for
// every tile shape.  The gate's weight gradient keeps its terms in LDS for other threads, so
// only the loads of its x tiles run here, for every block, stage and thread.
#include <random>
#include <vector>

#include "gemm2.hpp"
#include "gemm_f32.hpp"
#include "g2cfg.hpp"   // the launch helpers' tile shapes

thread_local hostcheck_dim3 threadIdx, blockIdx, gridDim, blockDim;
thread_local char* hostcheck_smem;
namespace dmoe {
void hostcheck_g2l(const void* g, char* l) { std::memcpy(l, g, 16); }
}
hostcheck_s16x4 hostcheck_lds_tr(const void* p) {
  hostcheck_s16x4 v;
  std::memcpy(&v, p, 8);
  return v;
}

using namespace dmoe;

template <typename T>
static T* buf(size_t n) { return static_cast<T*>(std::calloc(n ? n : 1, sizeof(T))); }

// tile plan as the tile_plan kernel writes it: m-tile prefix per expert, then the prefix
// of experts with rows
static std::vector<int32_t> plan_of(const std::vector<int32_t>& off, int N, int TMR) {
  std::vector<int32_t> plan(2 * (N + 1));
  int bm = 0, ba = 0;
  for (int e = 0; e < N; ++e) {
    plan[e] = bm;
    plan[N + 1 + e] = ba;
    const int c = off[e + 1] - off[e];
    bm += (c + TMR - 1) / TMR;
    ba += c > 0;
  }
  plan[N] = bm;
  plan[N + 1 + N] = ba;
  return plan;
}

static long launches = 0;
static size_t dw_short = 0, dw_short_f32 = 0;   // elements taken off the weight-gradient buffer (self-test)

// f() once for every thread of a launch, with an LDS of its own of exactly `lds` bytes
template <typename F>
static void each_thread(int grid, int NT, size_t lds, F&& f) {
  gridDim = {(unsigned)grid, 1, 1};
  blockDim = {(unsigned)NT, 1, 1};
  for (int b = 0; b < grid; ++b)
    for (int t = 0; t < NT; ++t) {
      blockIdx = {(unsigned)b, 0, 0};
      threadIdx = {(unsigned)t, 0, 0};
      hostcheck_smem = static_cast<char*>(std::malloc(lds));
      f();
      std::free(hostcheck_smem);
    }
  ++launches;
}

template <int GM, bool AT, bool BT, int EPI, int BM, int BN, int WM, int WN, int ST, int BK, int STO, int XB>
static void run(GemmArgs<bf16> p, int64_t tiles_ub) {
  if (tiles_ub <= 0) return;
  const int NT = 64 * WM * WN;
  const size_t lds = gemm2_lds_bytes<BM, BN, ST, AT, BT, BK, WM * WN, STO, XB>();
  const int grid = (int)std::min<int64_t>(tiles_ub, 256);    // one block per compute unit
  p.chunked = grid >= 8;
  each_thread(grid, NT, lds, [&] { grouped_gemm2<GM, AT, BT, EPI, BM, BN, WM, WN, ST, 1, BK, STO, XB>(p); });
}
template <int GM, bool AT, bool BT, int EPI, typename C>
static void run_f32(GemmArgs<float> p, int64_t tiles_ub) {
  if (tiles_ub <= 0) return;
  const int grid = (int)std::min<int64_t>(tiles_ub, 256);
  p.chunked = grid >= 8;
  each_thread(grid, 64 * C::WM * C::WN, gemm_f32_lds_bytes<C::BM, C::BN, C::ST>(),
              [&] { grouped_gemm_f32<GM, AT, BT, EPI, C::BM, C::BN, C::WM, C::WN, C::ST>(p); });
}

template <typename E = bf16>
static GemmArgs<E> args_m(const std::vector<int32_t>& off, const std::vector<int32_t>& plan, int scale, int N,
                             bool active) {
  GemmArgs<E> p{};
  p.offsets = off.data();
  p.tprefix = plan.data() + (active ? N + 1 : 0);
  p.tscale = scale;
  p.groups = N;
  return p;
}

// grouped GEMMs of one Linear layer [n_in -> n_out]: forward with bias (and the
// activation when act), data gradient, weight gradient (stored, or the SGD update)
template <typename C, typename CW>
static void layer(const std::vector<int32_t>& off, int N, int P, int n_in, int n_out, bool act) {
  const auto plan = plan_of(off, N, C::TMR);
  const int64_t mt_ub = (P + C::TMR - 1) / C::TMR + std::min<int64_t>(N, P);
  const int64_t active_ub = std::min<int64_t>(N, P);
  bf16* X = buf<bf16>((size_t)P * n_in);
  bf16* W = buf<bf16>((size_t)N * n_out * n_in);
  bf16* b = buf<bf16>((size_t)N * n_out);
  bf16* Hh = buf<bf16>((size_t)P * n_out);
  bf16* Aa = buf<bf16>((size_t)P * n_out);
  bf16* dY = buf<bf16>((size_t)P * n_out);
  bf16* dX = buf<bf16>((size_t)P * n_in);
  bf16* dW = buf<bf16>((size_t)N * n_out * n_in - dw_short);
  {   // forward: C[rows, n_out] = X W^T + b (h, and a = act(h))
    const int nt = (n_out + C::BN - 1) / C::BN;
    GemmArgs<bf16> p = args_m(off, plan, nt, N, false);
    p.A = X; p.lda = n_in; p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
    p.C = Hh; p.ldc = n_out; p.C2 = Aa; p.bias = b; p.bias_gstride = n_out; p.N = n_out; p.K = n_in;
    if (act) run<GROUP_M, false, false, EPI_BIAS_ACT, C::BM, C::BN, C::WM, C::WN, C::ST, C::BK, STORE_DIRECT, C::XB>(p, mt_ub * nt);
    else run<GROUP_M, false, false, EPI_BIAS, C::BM, C::BN, C::WM, C::WN, C::ST, C::BK, STORE_DIRECT, C::XB>(p, mt_ub * nt);
  }
  {   // data gradient: dX = dY W (W read N-contiguous); with act, times act'(h) of a layer of n_in outputs
    const int nt = (n_in + C::BN - 1) / C::BN;
    GemmArgs<bf16> p = args_m(off, plan, nt, N, false);
    p.A = dY; p.lda = n_out; p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
    p.C = dX; p.ldc = n_in; p.aux = X; p.N = n_in; p.K = n_out;
    if (act) run<GROUP_M, false, true, EPI_DACT, C::BM, C::BN, C::WM, C::WN, C::ST, C::BK, STORE_DIRECT, C::XB>(p, mt_ub * nt);
    else run<GROUP_M, false, true, EPI_STORE, C::BM, C::BN, C::WM, C::WN, C::ST, C::BK, STORE_DIRECT, C::XB>(p, mt_ub * nt);
  }
  {   // weight gradient dW_e = dY_e^T X_e, stored and as the SGD update of W
    const int mt = (n_out + CW::BM - 1) / CW::BM, nt = (n_in + CW::BN - 1) / CW::BN;
    GemmArgs<bf16> p = args_m(off, plan, mt * nt, N, true);
    p.A = dY; p.lda = n_out; p.B = X; p.ldb = n_in;
    p.C = dW; p.ldc = n_in; p.c_gstride = (int64_t)n_out * n_in; p.M = n_out; p.N = n_in;
    run<GROUP_K, true, true, EPI_STORE, CW::BM, CW::BN, CW::WM, CW::WN, CW::ST, CW::BK, CW::STO, 0>(p, active_ub * mt * nt);
    p.C = W; p.lr = 0.5f;
    run<GROUP_K, true, true, EPI_SGD, CW::BM, CW::BN, CW::WM, CW::WN, CW::ST, CW::BK, CW::STO, 0>(p, active_ub * mt * nt);
  }
  std::free(X); std::free(W); std::free(b); std::free(Hh); std::free(Aa);
  std::free(dY); std::free(dX); std::free(dW);
}

// the same launches of an fp32 layer; CW: the weight gradients' shape
template <typename C, typename CW>
static void layer_f32(const std::vector<int32_t>& off, int N, int P, int n_in, int n_out, bool act) {
  const auto plan = plan_of(off, N, C::TMR);
  const int64_t mt_ub = (P + C::TMR - 1) / C::TMR + std::min<int64_t>(N, P);
  const int64_t active_ub = std::min<int64_t>(N, P);
  float* X = buf<float>((size_t)P * n_in);
  float* W = buf<float>((size_t)N * n_out * n_in);
  float* b = buf<float>((size_t)N * n_out);
  float* Hh = buf<float>((size_t)P * n_out);
  float* Aa = buf<float>((size_t)P * n_out);
  float* dY = buf<float>((size_t)P * n_out);
  float* dX = buf<float>((size_t)P * n_in);
  float* dW = buf<float>((size_t)N * n_out * n_in - dw_short_f32);
  {
    const int nt = (n_out + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(off, plan, nt, N, false);
    p.A = X; p.lda = n_in; p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
    p.C = Hh; p.ldc = n_out; p.C2 = Aa; p.bias = b; p.bias_gstride = n_out; p.N = n_out; p.K = n_in;
    if (act) run_f32<GROUP_M, false, false, EPI_BIAS_ACT, C>(p, mt_ub * nt);
    else run_f32<GROUP_M, false, false, EPI_BIAS, C>(p, mt_ub * nt);
  }
  {
    const int nt = (n_in + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(off, plan, nt, N, false);
    p.A = dY; p.lda = n_out; p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
    p.C = dX; p.ldc = n_in; p.aux = X; p.N = n_in; p.K = n_out;
    if (act) run_f32<GROUP_M, false, true, EPI_DACT, C>(p, mt_ub * nt);
    else run_f32<GROUP_M, false, true, EPI_STORE, C>(p, mt_ub * nt);
  }
  {
    const int mt = (n_out + CW::BM - 1) / CW::BM, nt = (n_in + CW::BN - 1) / CW::BN;
    GemmArgs<float> p = args_m<float>(off, plan, mt * nt, N, true);
    p.A = dY; p.lda = n_out; p.B = X; p.ldb = n_in;
    p.C = dW; p.ldc = n_in; p.c_gstride = (int64_t)n_out * n_in; p.M = n_out; p.N = n_in;
    run_f32<GROUP_K, true, true, EPI_STORE, CW>(p, active_ub * mt * nt);
    p.C = W; p.lr = 0.5f;
    run_f32<GROUP_K, true, true, EPI_SGD, CW>(p, active_ub * mt * nt);
  }
  std::free(X); std::free(W); std::free(b); std::free(Hh); std::free(Aa);
  std::free(dY); std::free(dX); std::free(dW);
}

// The loads of x [T, D] in the gate's weight gradient: blocks of 128 columns and `split` tokens,
// stages of TOK tokens, four waves, the tile TX.
template <typename E, typename TX, int TOK>
static void gate_x_loads(int T, int D, int split) {
  E* x = buf<E>((size_t)T * D);
  const int nb = (D + 127) / 128, ns = (T + split - 1) / split;
  each_thread(nb * ns, 256, TX::BYTES, [&] {
    const int n0 = (int)(blockIdx.x % nb) * 128, tb = (int)(blockIdx.x / nb) * split, te = std::min(T, tb + split);
    const int nk = (te - tb + TOK - 1) / TOK;
    const E* at = x + (int64_t)tb * D + n0;
    for (int kt = 0; kt < nk; ++kt)
      TX::load(at + (int64_t)kt * TOK * D, D, D - n0, te - tb - kt * TOK, hostcheck_smem, (int)(threadIdx.x >> 6),
               (int)(threadIdx.x & 63));
  });
  std::free(x);
}

// row counts per expert: random around `mean`, expert 1 empty, expert 0 heavy
static std::vector<int32_t> offsets_of(int N, int mean, int spread, unsigned seed) {
  std::mt19937 rng(seed);
  std::vector<int32_t> off(N + 1, 0);
  for (int e = 0; e < N; ++e) {
    int c = mean - spread + (int)(rng() % (2 * spread + 1));
    if (e == 1) c = 0;
    if (e == 0) c = 2 * mean + spread;
    off[e + 1] = off[e] + std::max(c, 0);
  }
  return off;
}

int main(int argc, char** argv) {
  // "short": the weight-gradient buffer is 8 elements short, which the run must report
  if (argc > 1 && std::strcmp(argv[1], "short") == 0) dw_short = 8;
  if (argc > 1 && std::strcmp(argv[1], "short_f32") == 0) dw_short_f32 = 4;
  // (D, H): multiples of 64 as the API requires; one of them not a multiple of 256, so
  // the last column tile and the last m-tile of the weight gradients are partial
  {   // 256 x 256 tiles: experts around 288 rows (8- and 9-block tiles, some 3 m-tiles)
    const int N = 6;
    const auto off = offsets_of(N, 290, 40, 1);
    const int P = off[N];
    layer<G2Fat, G2DW>(off, N, P, 256, 320, true);
    layer<G2Fat, G2DW>(off, N, P, 320, 256, false);
    layer<G2Fat, G2DWShort>(off, N, P, 192, 256, true);
  }
  {   // 32 x 256 tiles: few rows per expert, 32-deep weight-gradient stages
    const int N = 12;
    const auto off = offsets_of(N, 19, 17, 2);
    const int P = off[N];
    layer<G2Skinny, G2DWShort>(off, N, P, 128, 320, true);
    layer<G2Skinny, G2DWShort>(off, N, P, 320, 128, false);
    layer<G2Skinny, G2DW>(off, N, P, 64, 256, false);
  }
  {   // the shapes between: row counts around their heights
    const auto few = offsets_of(12, 19, 17, 3), some = offsets_of(8, 64, 40, 4), many = offsets_of(6, 130, 100, 5);
    layer<G2Narrow, G2DWShort>(few, 12, few[12], 128, 320, true);
    layer<G2Narrow, G2DWShort>(few, 12, few[12], 320, 192, false);
    layer<G2Mid64, G2DW>(some, 8, some[8], 192, 320, true);
    layer<G2Mid64, G2DWShort>(some, 8, some[8], 320, 64, false);
    layer<G2Mid, G2DW>(many, 6, many[6], 192, 320, true);
    layer<G2Mid, G2DW>(many, 6, many[6], 320, 128, false);
  }
  {   // fp32
    const auto few = offsets_of(9, 19, 17, 6), some = offsets_of(7, 64, 40, 7);
    layer_f32<CfgF32Skinny, CfgF32>(few, 9, few[9], 64, 192, true);
    layer_f32<CfgF32Skinny, CfgF32>(few, 9, few[9], 192, 128, false);
    layer_f32<CfgF32, CfgF32DW>(some, 7, some[7], 192, 320, true);
    layer_f32<CfgF32, CfgF32DW>(some, 7, some[7], 320, 64, false);
  }
  // the tiles of the gate's weight gradient: half a column block, ragged stages and splits
  for (const int T : {1, 63, 65, 129, 321}) {
    gate_x_loads<bf16, NcTile<128, 4, 64>, 64>(T, 192, 128);
    gate_x_loads<bf16, NcTile<128, 4, 64>, 64>(T, 64, 320);
    gate_x_loads<float, NcTileF32<128, 4>, 32>(T, 192, 128);
    gate_x_loads<float, NcTileF32<128, 4>, 32>(T, 64, 320);
  }
  std::printf("gemm bounds: %ld launches checked\n", launches);
  return 0;
}
