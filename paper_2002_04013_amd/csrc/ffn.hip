// Expert feed-forward blocks on the per-expert row groups (the Runtime's batched
// Forward and Backward of Sec. 3.3), as grouped GEMMs on MFMA.
#include <algorithm>

#include "grouped.hpp"

namespace dmoe {

// h = x W1^T + b1, a = act(h); `up_only` for the recompute form of the backward, else also
// y = a W2^T + b2.  The plan's heights: (a) for the H columns of h, (b) for the D of y.
static void ffn_fwd_bf16(const Shape& s, const int32_t* offsets, const bf16* xp, const bf16* W1,
                         const bf16* b1, const bf16* W2, const bf16* b2, bf16* h, bf16* a, bf16* yp,
                         const Plan& pl, bool up_only, hipStream_t st) {
  const int N = (int)s.N, D = (int)s.D, H = (int)s.H;
  run_tile_plan(s, offsets, row_tile_rows(s, H), row_tile_rows(s, D), pl, st);
  {
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.a, 0, N);
    p.A = xp; p.lda = D;
    p.B = W1; p.ldb = D; p.b_gstride = (int64_t)H * D;
    p.C = h; p.ldc = H; p.C2 = a;
    p.bias = b1; p.bias_gstride = H;
    p.N = H; p.K = D; p.act = s.act;
    run_gemm2_rows<false, EPI_BIAS_ACT>(s, p, st);
  }
  if (up_only) return;
  {
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.b, 0, N);
    p.A = a; p.lda = H;
    p.B = W2; p.ldb = H; p.b_gstride = (int64_t)D * H;
    p.C = yp; p.ldc = D;
    p.bias = b2; p.bias_gstride = D;
    p.N = D; p.K = H; p.act = s.act;
    run_gemm2_rows<false, EPI_BIAS>(s, p, st);
  }
}

// SGD: dW1, db1, dW2, db2 are the parameters W1, b1, W2, b2 themselves, updated in place
// (W <- W - lr dW, b <- b - lr db) after their last use, the gradients never stored: dh reads
// W2 before W2's update, dx_perm reads W1 before W1's update.  planned: pl holds the plans of
// these offsets already (the recompute form's up-projection).
template <typename CW, bool SGD>
static void ffn_bwd_bf16(const Shape& s, const int32_t* offsets, const bf16* xp, const bf16* h,
                         const bf16* a, const bf16* dyp, const bf16* W1, const bf16* W2, bf16* dh, bf16* dxp,
                         bf16* dW1, bf16* db1, bf16* dW2, bf16* db2, const Plan& pl, bool planned, float lr,
                         hipStream_t st) {
  constexpr int EPI_W = SGD ? EPI_SGD : EPI_STORE;
  const int N = (int)s.N, D = (int)s.D, H = (int)s.H;
  const int64_t active_ub = std::min<int64_t>(s.N, s.P);
  if (!planned) run_tile_plan(s, offsets, row_tile_rows(s, H), row_tile_rows(s, D), pl, st);
  {   // dh = (dy W2) * act'(h): W2_e read as (n = h, k = d), N-contiguous
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.a, 0, N);
    p.A = dyp; p.lda = D;
    p.B = W2; p.ldb = H; p.b_gstride = (int64_t)D * H;
    p.C = dh; p.ldc = H; p.aux = h;
    p.N = H; p.K = D; p.act = s.act;
    run_gemm2_rows<true, EPI_DACT>(s, p, st);
  }
  {   // dW2_e = dy_e^T a_e   [D, H]
    const int mt = (D + CW::BM - 1) / CW::BM, nt = (H + CW::BN - 1) / CW::BN;
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.act, mt * nt, N);
    p.A = dyp; p.lda = D;
    p.B = a; p.ldb = H;
    p.C = dW2; p.ldc = H; p.c_gstride = (int64_t)D * H;
    p.M = D; p.N = H; p.act = s.act; p.lr = lr;
    run_gemm2<GROUP_K, true, true, EPI_W, CW::BM, CW::BN, CW::WM, CW::WN, CW::ST, CW::BK, CW::STO>(p, active_ub * mt * nt, st);
  }
  {   // dx_perm = dh W1: W1_e read as (n = d, k = h), N-contiguous
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.b, 0, N);
    p.A = dh; p.lda = H;
    p.B = W1; p.ldb = D; p.b_gstride = (int64_t)H * D;
    p.C = dxp; p.ldc = D;
    p.N = D; p.K = H; p.act = s.act;
    run_gemm2_rows<true, EPI_STORE>(s, p, st);
  }
  {   // dW1_e = dh_e^T x_e   [H, D]
    const int mt = (H + CW::BM - 1) / CW::BM, nt = (D + CW::BN - 1) / CW::BN;
    GemmArgs<bf16> p = args_m<bf16>(offsets, pl.act, mt * nt, N);
    p.A = dh; p.lda = H;
    p.B = xp; p.ldb = D;
    p.C = dW1; p.ldc = D; p.c_gstride = (int64_t)H * D;
    p.M = H; p.N = D; p.act = s.act; p.lr = lr;
    run_gemm2<GROUP_K, true, true, EPI_W, CW::BM, CW::BN, CW::WM, CW::WN, CW::ST, CW::BK, CW::STO>(p, active_ub * mt * nt, st);
  }
  run_colsum<bf16, SGD>(s, offsets, dh, H, db1, dyp, D, db2, lr, st);
}

template <typename C>
static void ffn_fwd_f32(const Shape& s, const int32_t* offsets, const float* xp, const float* W1,
                        const float* b1, const float* W2, const float* b2, float* h, float* a, float* yp,
                        const Plan& pl, hipStream_t st) {
  const int N = (int)s.N, D = (int)s.D, H = (int)s.H;
  const int64_t mt_ub = (s.P + C::TMR - 1) / C::TMR + std::min<int64_t>(s.N, s.P);
  run_tile_plan(s, offsets, C::TMR, C::TMR, pl, st);
  // h = x W1^T + b1, a = act(h)
  {
    const int nt = (H + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.a, nt, N);
    p.A = xp; p.lda = D;
    p.B = W1; p.ldb = D; p.b_gstride = (int64_t)H * D;
    p.C = h; p.ldc = H; p.C2 = a;
    p.bias = b1; p.bias_gstride = H;
    p.N = H; p.K = D; p.act = s.act;
    run_gemm_f32<GROUP_M, false, false, EPI_BIAS_ACT, C>(p, mt_ub * nt, st);
  }
  // y = a W2^T + b2
  {
    const int nt = (D + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.a, nt, N);
    p.A = a; p.lda = H;
    p.B = W2; p.ldb = H; p.b_gstride = (int64_t)D * H;
    p.C = yp; p.ldc = D;
    p.bias = b2; p.bias_gstride = D;
    p.N = D; p.K = H; p.act = s.act;
    run_gemm_f32<GROUP_M, false, false, EPI_BIAS, C>(p, mt_ub * nt, st);
  }
}

// SGD: dW1, db1, dW2, db2 are the parameters W1, b1, W2, b2 themselves, updated in
// place (W <- W - lr dW) after their last read: dh reads W2 before W2's update and
// dx_perm reads W1 before W1's update.
template <typename C, typename CW, bool SGD = false>
static void ffn_bwd_f32(const Shape& s, const int32_t* offsets, const float* xp, const float* h,
                        const float* a, const float* dyp, const float* W1, const float* W2, float* dh, float* dxp,
                        float* dW1, float* db1, float* dW2, float* db2, const Plan& pl, bool planned, float lr,
                        hipStream_t st) {
  constexpr int EPI_W = SGD ? EPI_SGD : EPI_STORE;
  const int N = (int)s.N, D = (int)s.D, H = (int)s.H;
  const int64_t mt_ub = (s.P + C::TMR - 1) / C::TMR + std::min<int64_t>(s.N, s.P);
  const int64_t active_ub = std::min<int64_t>(s.N, s.P);
  if (!planned) run_tile_plan(s, offsets, C::TMR, C::TMR, pl, st);
  // dh = (dy W2) * act'(h)       B = W2_e viewed as (n = h, k = d): N-contiguous
  {
    const int nt = (H + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.a, nt, N);
    p.A = dyp; p.lda = D;
    p.B = W2; p.ldb = H; p.b_gstride = (int64_t)D * H;
    p.C = dh; p.ldc = H; p.aux = h;
    p.N = H; p.K = D; p.act = s.act;
    run_gemm_f32<GROUP_M, false, true, EPI_DACT, C>(p, mt_ub * nt, st);
  }
  // dW2_e = dy_e^T a_e   [D, H]
  {
    const int mt = (D + CW::BM - 1) / CW::BM, nt = (H + CW::BN - 1) / CW::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.act, mt * nt, N);
    p.A = dyp; p.lda = D;
    p.B = a; p.ldb = H;
    p.C = dW2; p.ldc = H; p.c_gstride = (int64_t)D * H;
    p.M = D; p.N = H; p.act = s.act; p.lr = lr;
    run_gemm_f32<GROUP_K, true, true, EPI_W, CW>(p, active_ub * mt * nt, st);
  }
  // dx_perm = dh W1              B = W1_e viewed as (n = d, k = h): N-contiguous
  {
    const int nt = (D + C::BN - 1) / C::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.a, nt, N);
    p.A = dh; p.lda = H;
    p.B = W1; p.ldb = D; p.b_gstride = (int64_t)H * D;
    p.C = dxp; p.ldc = D;
    p.N = D; p.K = H; p.act = s.act;
    run_gemm_f32<GROUP_M, false, true, EPI_STORE, C>(p, mt_ub * nt, st);
  }
  // dW1_e = dh_e^T x_e   [H, D]
  {
    const int mt = (H + CW::BM - 1) / CW::BM, nt = (D + CW::BN - 1) / CW::BN;
    GemmArgs<float> p = args_m<float>(offsets, pl.act, mt * nt, N);
    p.A = dh; p.lda = H;
    p.B = xp; p.ldb = D;
    p.C = dW1; p.ldc = D; p.c_gstride = (int64_t)H * D;
    p.M = H; p.N = D; p.act = s.act; p.lr = lr;
    run_gemm_f32<GROUP_K, true, true, EPI_W, CW>(p, active_ub * mt * nt, st);
  }
  run_colsum<float, SGD>(s, offsets, dh, H, db1, dyp, D, db2, lr, st);   // bias gradients
}

template <typename C>
static void ffn_up_f32(const Shape& s, const int32_t* offsets, const float* xp, const float* W1, const float* b1, float* h, float* a,
                       const Plan& pl, hipStream_t st) {
  const int N = (int)s.N, D = (int)s.D, H = (int)s.H;
  const int64_t mt_ub = (s.P + C::TMR - 1) / C::TMR + std::min<int64_t>(s.N, s.P);
  run_tile_plan(s, offsets, C::TMR, C::TMR, pl, st);
  const int nt = (H + C::BN - 1) / C::BN;
  GemmArgs<float> p = args_m<float>(offsets, pl.a, nt, N);
  p.A = xp; p.lda = D;
  p.B = W1; p.ldb = D; p.b_gstride = (int64_t)H * D;
  p.C = h; p.ldc = H; p.C2 = a;
  p.bias = b1; p.bias_gstride = H;
  p.N = H; p.K = D; p.act = s.act;
  run_gemm_f32<GROUP_M, false, false, EPI_BIAS_ACT, C>(p, mt_ub * nt, st);
}

// The forward on tile plans at pl (2 (N + 1) ints of device memory).
static int ffn_fwd_impl(const Shape& s, const int32_t* offsets, const void* x_perm, const void* W1,
                        const void* b1, const void* W2, const void* b2, void* h, void* a, void* y_perm,
                        const Plan& pl, hipStream_t st) {
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    ffn_fwd_bf16(s, offsets, c(x_perm), c(W1), c(b1), c(W2), c(b2), m(h), m(a), m(y_perm), pl, false, st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    if (use_fat_f32(s))
      ffn_fwd_f32<CfgF32>(s, offsets, c(x_perm), c(W1), c(b1), c(W2), c(b2), m(h), m(a), m(y_perm), pl, st);
    else
      ffn_fwd_f32<CfgF32Skinny>(s, offsets, c(x_perm), c(W1), c(b1), c(W2), c(b2), m(h), m(a), m(y_perm), pl, st);
  }
  return launch_status();
}

static int ffn_fwd_check(const dmoe_dims* dims, Shape* s, const int32_t* offsets, const void* x_perm, const void* W1,
                         const void* b1, const void* W2, const void* b2, const void* h, const void* a,
                         const void* y_perm) {
  const int rc = check_dims(dims, s);
  if (rc) return rc;
  if (s->T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !W1 || !b1 || !W2 || !b2 || !h || !a || !y_perm) return DMOE_EINVAL;
  for (const void* q : {x_perm, W1, W2, h, a, y_perm})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  return DMOE_OK;
}

// Scratch of dmoe_expert_ffn_fwd_noalloc: the two tile plans, 2 (N + 1) ints for N <= NMAX.
// Each device holds its own copy; host code reaches it only through the address
// hipGetSymbolAddress returns on that device (the array's name is no device address
// in host code).
constexpr size_t FFN_SCRATCH_BYTES = ((size_t)2 * (NMAX + 1) * sizeof(int32_t) + 255) & ~(size_t)255;
static __device__ __align__(256) unsigned char scratch[FFN_SCRATCH_BYTES];

// scratch's address on the current device, looked up on the first call there.
static int32_t* scratch_on_device() {
  static std::atomic<void*> addr[MAX_DEVICES];
  const int dev = current_device();
  if (dev < 0) return nullptr;
  void* p = addr[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    addr[dev].store(p, std::memory_order_release);
  }
  return reinterpret_cast<int32_t*>(p);
}

}  // namespace dmoe

using namespace dmoe;

extern "C" int dmoe_expert_ffn_fwd(const dmoe_dims* dims, const int32_t* offsets, const void* x_perm,
                                   const void* W1, const void* b1, const void* W2, const void* b2,
                                   void* h, void* a, void* y_perm, void* ws, void* stream) {
  Shape s;
  int rc = ffn_fwd_check(dims, &s, offsets, x_perm, W1, b1, W2, b2, h, a, y_perm);
  if (rc || s.T == 0) return rc;
  if (!ws) return DMOE_EINVAL;
  if (!aligned16(ws)) return DMOE_EUNSUPPORTED;
  const Workspace L = workspace_layout(s);
  int32_t* tpre = reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + L.tiles_off);
  return ffn_fwd_impl(s, offsets, x_perm, W1, b1, W2, b2, h, a, y_perm, plan_at(tpre, s.N, false),
                      reinterpret_cast<hipStream_t>(stream));
}

extern "C" int dmoe_expert_ffn_fwd_noalloc(const dmoe_dims* dims, const int32_t* offsets, const void* x_perm,
                                           const void* W1, const void* b1, const void* W2, const void* b2,
                                           void* h, void* a, void* y_perm, void* stream) {
  Shape s;
  int rc = ffn_fwd_check(dims, &s, offsets, x_perm, W1, b1, W2, b2, h, a, y_perm);
  if (rc || s.T == 0) return rc;
  if ((size_t)2 * (s.N + 1) * sizeof(int32_t) > FFN_SCRATCH_BYTES) return DMOE_EUNSUPPORTED;
  int32_t* tpre = scratch_on_device();
  if (!tpre) return DMOE_EHIP;
  return ffn_fwd_impl(s, offsets, x_perm, W1, b1, W2, b2, h, a, y_perm, plan_at(tpre, s.N, false),
                      reinterpret_cast<hipStream_t>(stream));
}

// planned: the workspace holds the tile plans of these offsets already.
static int ffn_bwd_checked(const dmoe_dims* dims, const int32_t* offsets, const int32_t* counts,
                           const void* x_perm, const void* h, const void* a, const void* dy_perm, const void* W1,
                           const void* W2, void* dh, void* dx_perm, void* dW1, void* db1, void* dW2, void* db2,
                           void* ws, bool planned, void* stream) {
  (void)counts;
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !h || !a || !dy_perm || !W1 || !W2 || !dh || !dx_perm || !dW1 || !db1 ||
      !dW2 || !db2 || !ws)
    return DMOE_EINVAL;
  for (const void* q : {x_perm, h, a, dy_perm, W1, W2, (const void*)dh, (const void*)dx_perm,
                        (const void*)dW1, (const void*)db1, (const void*)dW2, (const void*)db2, (const void*)ws})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  const Workspace L = workspace_layout(s);
  const Plan pl = plan_at(reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + L.tiles_off), s.N, true);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    if (deep_wgrad(s))
      ffn_bwd_bf16<G2DW, false>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh), m(dx_perm),
                                m(dW1), m(db1), m(dW2), m(db2), pl, planned, 0.f, st);
    else
      ffn_bwd_bf16<G2DWShort, false>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh), m(dx_perm),
                                     m(dW1), m(db1), m(dW2), m(db2), pl, planned, 0.f, st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    if (use_fat_f32(s))
      ffn_bwd_f32<CfgF32, CfgF32DW>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh), m(dx_perm),
                                  m(dW1), m(db1), m(dW2), m(db2), pl, planned, 0.f, st);
    else
      ffn_bwd_f32<CfgF32Skinny, CfgF32>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh),
                                        m(dx_perm), m(dW1), m(db1), m(dW2), m(db2), pl, planned, 0.f, st);
  }
  return launch_status();
}

extern "C" int dmoe_expert_ffn_bwd(const dmoe_dims* dims, const int32_t* offsets, const int32_t* counts,
                                   const void* x_perm, const void* h, const void* a, const void* dy_perm,
                                   const void* W1, const void* W2, void* dh, void* dx_perm, void* dW1,
                                   void* db1, void* dW2, void* db2, void* ws, void* stream) {
  return ffn_bwd_checked(dims, offsets, counts, x_perm, h, a, dy_perm, W1, W2, dh, dx_perm, dW1, db1, dW2, db2, ws,
                         false, stream);
}

extern "C" int dmoe_expert_ffn_bwd_recompute(const dmoe_dims* dims, const int32_t* offsets, const int32_t* counts,
                                             const void* x_perm, const void* W1, const void* b1, const void* W2,
                                             const void* dy_perm, void* h, void* a, void* dx_perm, void* dW1,
                                             void* db1, void* dW2, void* db2, void* ws, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !W1 || !b1 || !W2 || !dy_perm || !h || !a || !dx_perm || !dW1 || !db1 || !dW2 ||
      !db2 || !ws)
    return DMOE_EINVAL;
  for (const void* q : {x_perm, W1, W2, dy_perm, (const void*)h, (const void*)a, (const void*)dx_perm,
                        (const void*)dW1, (const void*)db1, (const void*)dW2, (const void*)db2, (const void*)ws})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  const Workspace L = workspace_layout(s);
  const Plan pl = plan_at(reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + L.tiles_off), s.N, true);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // 1. recompute the up-projection of the forward into the scratch h and a
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    ffn_fwd_bf16(s, offsets, c(x_perm), c(W1), c(b1), nullptr, nullptr, m(h), m(a), nullptr, pl, true, st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    if (use_fat_f32(s)) ffn_up_f32<CfgF32>(s, offsets, c(x_perm), c(W1), c(b1), m(h), m(a), pl, st);
    else ffn_up_f32<CfgF32Skinny>(s, offsets, c(x_perm), c(W1), c(b1), m(h), m(a), pl, st);
  }
  // 2. the backward proper, dh written over h
  return ffn_bwd_checked(dims, offsets, counts, x_perm, h, a, dy_perm, W1, W2, h, dx_perm, dW1, db1, dW2, db2, ws,
                         true, stream);
}

extern "C" int dmoe_expert_ffn_bwd_sgd(const dmoe_dims* dims, const int32_t* offsets, const int32_t* counts,
                                       const void* x_perm, const void* h, const void* a, const void* dy_perm,
                                       void* W1, void* b1, void* W2, void* b2, float lr, void* dh, void* dx_perm,
                                       void* ws, void* stream) {
  (void)counts;
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !h || !a || !dy_perm || !W1 || !b1 || !W2 || !b2 || !dh || !dx_perm || !ws)
    return DMOE_EINVAL;
  if (!(lr == lr)) return DMOE_EINVAL;                       // NaN step size
  for (const void* q : {x_perm, h, a, dy_perm, (const void*)W1, (const void*)b1, (const void*)W2,
                        (const void*)b2, (const void*)dh, (const void*)dx_perm, (const void*)ws})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  const Workspace L = workspace_layout(s);
  const Plan pl = plan_at(reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + L.tiles_off), s.N, true);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    if (deep_wgrad(s))
      ffn_bwd_bf16<G2DW, true>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh), m(dx_perm),
                               m(W1), m(b1), m(W2), m(b2), pl, false, lr, st);
    else
      ffn_bwd_bf16<G2DWShort, true>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh), m(dx_perm),
                                    m(W1), m(b1), m(W2), m(b2), pl, false, lr, st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    if (use_fat_f32(s))
      ffn_bwd_f32<CfgF32, CfgF32DW, true>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh),
                                        m(dx_perm), m(W1), m(b1), m(W2), m(b2), pl, false, lr, st);
    else
      ffn_bwd_f32<CfgF32Skinny, CfgF32, true>(s, offsets, c(x_perm), c(h), c(a), c(dy_perm), c(W1), c(W2), m(dh),
                                              m(dx_perm), m(W1), m(b1), m(W2), m(b2), pl, false, lr, st);
  }
  return launch_status();
}
