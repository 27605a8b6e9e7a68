// The feed-forward block expert of Sec. 4.1 on the per-expert row groups: three
// linear layers with layer normalisation and an activation between them,
//   h1 = x W1^T + b1, a1 = act(LN(h1; g1, be1)), h2 = a1 W2^T + b2,
//   a2 = act(LN(h2; g2, be2)), y = a2 W3^T + b3,
// LN(h; g, b) = g (h - mean) / sqrt(var + eps) + b over the F features of a row
// (biased variance, eps = 1e-5).  The linear layers run on the grouped GEMMs; the
// normalisation, its affine map and the activation are one row kernel.  The backward of
// that step inside the block is one pass over its rows (ln_bwd_kernel), with a reduction
// of the column sums that its blocks share; the step's own entry point, which has no
// workspace for those, takes a row kernel (input gradient) and a per-expert column
// reduction (scale and shift gradients).
#include "grouped.hpp"

namespace dmoe {

constexpr float LN_EPS = 1e-5f;
constexpr int LN_NT = 256;       // 4 waves; a wave normalises one row at a time
constexpr int LN_CHMAX = 8;      // 16-byte chunks per lane: rows of up to 64*8*VEC values

// Expert that owns row r: the first e with offsets[e + 1] > r.
__device__ __forceinline__ int row_expert(const int32_t* offsets, int N, int r) {
  int lo = 0, hi = N - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid + 1] > r) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// fp32 layers use the library's erf; bf16 layers (outputs rounded to 2^-9) the
// erfc-based forms of common.hpp.
// ACT is the activation (DMOE_RELU or DMOE_GELU), fixed at compile time.
template <typename E, int ACT> __device__ __forceinline__ float act_f(float z) {
  if constexpr (sizeof(E) == 4) return act_fwd(z, ACT);
  else return act_fwd_fast(z, ACT);
}
template <typename E, int ACT> __device__ __forceinline__ float act_b(float z) {
  if constexpr (sizeof(E) == 4) return act_bwd(z, ACT);
  else return act_bwd_fast(z, ACT);
}

// Contiguous share of the rows [0, offsets[N]) for wave gw of nw.
struct RowRange { int r0, r1; };
__device__ __forceinline__ RowRange wave_rows(const int32_t* offsets, int N) {
  const int nw = gridDim.x * (LN_NT / 64);
  // the wave index through readfirstlane: every value derived from it is wave-uniform,
  // so row bounds, the row's expert and its statistics come from scalar loads, whose
  // waits do not include the wave's outstanding vector loads and stores
  const int gw = blockIdx.x * (LN_NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int P = offsets[N];
  const int per = (P + nw - 1) / nw;
  const int r0 = min(P, gw * per);
  return {r0, min(P, r0 + per)};
}

// a = act(g (h - mean) rstd + b) per row, stats[r] = (mean, rstd), g and b of the
// row's expert.  Lane l holds chunks l, l + 64, ... of the row (16 bytes each).  The
// next row is loaded before this row's results are stored (vector-memory operations
// retire in order, so a row's loads then never wait for the previous row's stores),
// and the expert's g and b stay in registers until the expert changes.
template <typename E, int CH, int ACT>
__global__ void __launch_bounds__(LN_NT)
ln_act_fwd_kernel(const E* h, const int32_t* offsets, int N, int F, const E* gamma, const E* beta,
                  E* a, float* stats) {
  constexpr int VEC = Vec<E>::N;
  const int lane = threadIdx.x & 63;
  const RowRange rr = wave_rows(offsets, N);
  if (rr.r0 >= rr.r1) return;
  const int nch = F / VEC;
  const float invF = 1.f / (float)F;
  int e = row_expert(offsets, N, rr.r0);
  int eend = offsets[e + 1];
  int eg = -1;                                   // expert whose g, b are in gv, bv
  uint4 hv[CH], gv[CH], bv[CH];
  auto load_row = [&](uint4 (&v)[CH], const E* src) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = lane + 64 * i;
      v[i] = c < nch ? *reinterpret_cast<const uint4*>(src + c * VEC) : make_uint4(0, 0, 0, 0);
    }
  };
  load_row(hv, h + (int64_t)rr.r0 * F);
  for (int r = rr.r0; r < rr.r1; ++r) {
    while (r >= eend) eend = offsets[++e + 1];
    if (e != eg) {
      load_row(gv, gamma + (int64_t)e * F);
      load_row(bv, beta + (int64_t)e * F);
      eg = e;
    }
    uint4 hn[CH];
    if (r + 1 < rr.r1) load_row(hn, h + (int64_t)(r + 1) * F);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      float x[VEC];
      Vec<E>::unpack(hv[i], x);
#pragma unroll
      for (int j = 0; j < VEC; ++j) s += x[j];
    }
    const float mean = wave_sum(s) * invF;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      if (lane + 64 * i >= nch) continue;
      float x[VEC];
      Vec<E>::unpack(hv[i], x);
#pragma unroll
      for (int j = 0; j < VEC; ++j) q += (x[j] - mean) * (x[j] - mean);
    }
    const float rstd = 1.f / sqrtf(wave_sum(q) * invF + LN_EPS);
    E* ar = a + (int64_t)r * F;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = lane + 64 * i;
      if (c >= nch) continue;
      float x[VEC], g[VEC], b[VEC], o[VEC];
      Vec<E>::unpack(hv[i], x);
      Vec<E>::unpack(gv[i], g);
      Vec<E>::unpack(bv[i], b);
#pragma unroll
      for (int j = 0; j < VEC; ++j) o[j] = act_f<E, ACT>(fmaf(g[j], (x[j] - mean) * rstd, b[j]));
      *reinterpret_cast<uint4*>(ar + c * VEC) = Vec<E>::pack(o);
    }
    if (lane == 0) *reinterpret_cast<float2*>(stats + 2 * (int64_t)r) = make_float2(mean, rstd);
    if (r + 1 < rr.r1) {
#pragma unroll
      for (int i = 0; i < CH; ++i) hv[i] = hn[i];
    }
  }
}

// Input gradient of the normalisation step, per row:
//   n = (h - mean) rstd, z = g n + b, dn = da act'(z) g,
//   dh = rstd (dn - mean_f(dn) - n mean_f(dn n)).
// The whole row is read before it is written, so dh may alias da.  dn is kept in fp32
// registers between the two passes (the second pass only recomputes n); g and b are
// read per chunk (the expert's two rows stay in L1), so that several waves share a
// SIMD and one wave's arithmetic covers another's loads.
template <typename E, int CH, int ACT>
__global__ void __launch_bounds__(LN_NT)
ln_act_bwd_rows_kernel(const E* h, const float* stats, const int32_t* offsets, int N, int F, const E* gamma,
                       const E* beta, const E* da, E* dh) {
  constexpr int VEC = Vec<E>::N;
  const int lane = threadIdx.x & 63;
  const RowRange rr = wave_rows(offsets, N);
  if (rr.r0 >= rr.r1) return;
  const int nch = F / VEC;
  const float invF = 1.f / (float)F;
  int e = row_expert(offsets, N, rr.r0);
  int eend = offsets[e + 1];
  for (int r = rr.r0; r < rr.r1; ++r) {
    while (r >= eend) eend = offsets[++e + 1];
    const E* gr = gamma + (int64_t)e * F;
    const E* br = beta + (int64_t)e * F;
    uint4 hv[CH], dv[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = lane + 64 * i;
      hv[i] = c < nch ? *reinterpret_cast<const uint4*>(h + (int64_t)r * F + c * VEC) : make_uint4(0, 0, 0, 0);
      dv[i] = c < nch ? *reinterpret_cast<const uint4*>(da + (int64_t)r * F + c * VEC) : make_uint4(0, 0, 0, 0);
    }
    const float2 st = *reinterpret_cast<const float2*>(stats + 2 * (int64_t)r);
    const float mean = st.x, rstd = st.y;
    float dnf[CH][VEC];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = lane + 64 * i;
#pragma unroll
      for (int j = 0; j < VEC; ++j) dnf[i][j] = 0.f;
      if (c >= nch) continue;
      const uint4 gq = *reinterpret_cast<const uint4*>(gr + c * VEC);
      const uint4 bq = *reinterpret_cast<const uint4*>(br + c * VEC);
      float x[VEC], d[VEC], g[VEC], b[VEC];
      Vec<E>::unpack(hv[i], x);
      Vec<E>::unpack(dv[i], d);
      Vec<E>::unpack(gq, g);
      Vec<E>::unpack(bq, b);
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const float n = (x[j] - mean) * rstd;
        const float dn = d[j] * act_b<E, ACT>(fmaf(g[j], n, b[j])) * g[j];
        dnf[i][j] = dn;
        s1 += dn;
        s2 += dn * n;
      }
    }
    const float m1 = wave_sum(s1) * invF, m2 = wave_sum(s2) * invF;
    E* out = dh + (int64_t)r * F;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = lane + 64 * i;
      if (c >= nch) continue;
      float x[VEC], o[VEC];
      Vec<E>::unpack(hv[i], x);
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const float n = (x[j] - mean) * rstd;
        o[j] = rstd * (dnf[i][j] - m1 - n * m2);
      }
      *reinterpret_cast<uint4*>(out + c * VEC) = Vec<E>::pack(o);
    }
  }
}

// Scale and shift gradients of the normalisation step, per expert e and feature f:
//   dgamma[e][f] = sum over e's rows of da act'(z) n,  dbeta[e][f] = sum of da act'(z).
// Block (x, e) takes CL * VEC features of expert e, its rows split over slices as in
// segment_colsum (64 experts of 2048 rows, F = 4096 bf16: 722-784 -> 390-410 us).
// Experts without rows are left untouched.
template <typename E, int ACT, int CL>
__global__ void __launch_bounds__(CS_NT)
ln_act_bwd_params_kernel(const E* h, const float* stats, const int32_t* offsets, int F, const E* gamma,
                         const E* beta, const E* da, E* dgamma, E* dbeta) {
  constexpr int VEC = Vec<E>::N, S = CS_NT / CL;
  const int e = blockIdx.y;
  const int r0 = offsets[e], r1 = offsets[e + 1];
  if (r1 == r0) return;
  const int c = ((int)blockIdx.x * CL + (int)threadIdx.x % CL) * VEC;
  const bool cok = c < F;
  const int cc = cok ? c : 0;
  float g[VEC], b[VEC], acc[2][VEC];                  // acc: scale, shift
  Vec<E>::unpack(*reinterpret_cast<const uint4*>(gamma + (int64_t)e * F + cc), g);
  Vec<E>::unpack(*reinterpret_cast<const uint4*>(beta + (int64_t)e * F + cc), b);
#pragma unroll
  for (int j = 0; j < VEC; ++j) acc[0][j] = acc[1][j] = 0.f;
  auto add = [&](const uint4& hv, const uint4& dv, const float2& st) {
    float x[VEC], d[VEC];
    Vec<E>::unpack(hv, x);
    Vec<E>::unpack(dv, d);
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
      const float n = (x[j] - st.x) * st.y;
      const float dz = d[j] * act_b<E, ACT>(fmaf(g[j], n, b[j]));
      acc[0][j] += dz * n;
      acc[1][j] += dz;
    }
  };
  constexpr int U = 4;
  if (S == 1 && !cok) return;
  int r = S == 1 ? r0 : cok ? r0 + (int)threadIdx.x / CL : r1;      // as in segment_colsum
  for (; r + (U - 1) * S < r1; r += U * S) {
    uint4 hv[U], dv[U];
    float2 st[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t ru = r + u * S;
      hv[u] = *reinterpret_cast<const uint4*>(h + ru * F + cc);
      dv[u] = *reinterpret_cast<const uint4*>(da + ru * F + cc);
      st[u] = *reinterpret_cast<const float2*>(stats + 2 * ru);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) add(hv[u], dv[u], st[u]);
  }
  for (; r < r1; r += S)
    add(*reinterpret_cast<const uint4*>(h + (int64_t)r * F + cc), *reinterpret_cast<const uint4*>(da + (int64_t)r * F + cc),
        *reinterpret_cast<const float2*>(stats + 2 * (int64_t)r));
  colsum_slices<CL>(acc);
  if ((int)threadIdx.x >= CL || !cok) return;
  *reinterpret_cast<uint4*>(dgamma + (int64_t)e * F + c) = Vec<E>::pack(acc[0]);
  *reinterpret_cast<uint4*>(dbeta + (int64_t)e * F + c) = Vec<E>::pack(acc[1]);
}

// ---- the whole backward of a normalisation step in one pass over h and da ----
//
// ln_bwd_kernel does what ln_act_bwd_rows_kernel, ln_act_bwd_params_kernel and the column sum
// of dh (the bias gradient of the linear layer before it) do: dh per row, and per expert
// dgamma, dbeta and db = sum of its dh rows (as stored).  A block holds whole rows, one
// 16-byte chunk to a thread, two rows at a time with the next two loaded ahead; the row sums
// meet in LDS, the column sums stay in the thread's registers while the expert's rows last.
// A block takes a contiguous share of all rows: the sums of an expert that lies in one block
// are stored at once, the pieces of an expert spread over several go to `part` and
// ln_bwd_reduce_kernel adds them in row order.
// Bound by memory: h and da read, dh written.  64 experts of 2048 rows, F = 4096 bf16: 711 to
// 749 us (4.5 TB/s) and 9 for the reduction, in place of 390 (parameters) + 684 (rows) + 231
// (column sums), which read h and da twice and dh once more.  Held to 128 registers, for two
// blocks to a unit, it spills and takes 1590 us.
constexpr int LB_R = 2;                  // rows in flight per block step

static int lb_threads(int64_t chunks) { return chunks <= 64 ? 64 : chunks <= 128 ? 128 : chunks <= 256 ? 256 : 512; }
// `part` rows of 3 F floats: piece of the expert that begins in an earlier block: the block's
// index; piece of one that ends in a later block: after those, by expert or by block,
// whichever are fewer
__device__ __forceinline__ int lb_first_slot(int b) { return b; }
__device__ __forceinline__ int lb_last_slot(int nb, int N, int b, int e) { return nb + (N < nb ? e : b); }

// sum over the wave, left in lane 63
template <int CTRL, int ROWS>
__device__ __forceinline__ float add_dpp(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_sum63(float v) {
  v = add_dpp<0xB1, 0xf>(v);       // quad_perm [1,0,3,2]
  v = add_dpp<0x4E, 0xf>(v);       // quad_perm [2,3,0,1]
  v = add_dpp<0x141, 0xf>(v);      // row_half_mirror
  v = add_dpp<0x140, 0xf>(v);      // row_mirror: every lane holds its row's sum
  v = add_dpp<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
  v = add_dpp<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
  return v;
}

template <typename E, int ACT, int NT>
__global__ void __launch_bounds__(NT)
ln_bwd_kernel(const E* h, const float* stats, const int32_t* offsets, int N, int F, const E* gamma, const E* beta,
              const E* da, E* dh, E* dgamma, E* dbeta, E* db, float* part) {
  constexpr int VEC = Vec<E>::N, NW = NT / 64;
  __shared__ __align__(16) float red[2][NW][2 * LB_R];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = gridDim.x, blk = blockIdx.x;
  const int P = offsets[N];
  const int per = (P + nb - 1) / nb;
  const int r0 = min(P, blk * per), r1 = min(P, r0 + per);
  if (r0 >= r1) return;
  const bool on = tid * VEC < F;
  const int c = on ? tid * VEC : 0;
  const float invF = 1.f / (float)F;
  int e = row_expert(offsets, N, r0);
  int buf = 0;
  for (int r = r0; r < r1;) {
    while (offsets[e + 1] <= r) ++e;
    const int ebeg = offsets[e], eend = offsets[e + 1];
    const int pend = min(r1, eend);
    const uint4 gq = *reinterpret_cast<const uint4*>(gamma + (int64_t)e * F + c);
    const uint4 bq = *reinterpret_cast<const uint4*>(beta + (int64_t)e * F + c);
    float ag[VEC], ab[VEC], ad[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) ag[j] = ab[j] = ad[j] = 0.f;
    struct Rows { uint4 h[LB_R], d[LB_R]; float2 st[LB_R]; };
    Rows cur, nxt;
    auto load = [&](Rows& v, int q) {
#pragma unroll
      for (int u = 0; u < LB_R; ++u) {
        const int64_t row = min(q + u, pend - 1);
        v.h[u] = *reinterpret_cast<const uint4*>(h + row * F + c);
        v.d[u] = *reinterpret_cast<const uint4*>(da + row * F + c);
        v.st[u] = *reinterpret_cast<const float2*>(stats + 2 * row);
      }
    };
    load(cur, r);
    for (int q = r; q < pend; q += LB_R) {
      if (q + LB_R < pend) load(nxt, q + LB_R);
      float dn[LB_R][VEC];
      float s[2 * LB_R];
      float g[VEC], b[VEC];
      Vec<E>::unpack(gq, g);
      Vec<E>::unpack(bq, b);
#pragma unroll
      for (int u = 0; u < LB_R; ++u) {
        // a row past the piece contributes nothing (and is not stored below)
        const float live = on && q + u < pend ? 1.f : 0.f;
        float x[VEC], d[VEC];
        Vec<E>::unpack(cur.h[u], x);
        Vec<E>::unpack(cur.d[u], d);
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
          const float n = (x[j] - cur.st[u].x) * cur.st[u].y;
          const float dz = d[j] * act_b<E, ACT>(fmaf(g[j], n, b[j]));
          dn[u][j] = dz * g[j];
          s1 += dn[u][j];
          s2 += dn[u][j] * n;
          if (live != 0.f) { ag[j] += dz * n; ab[j] += dz; }
        }
        s[2 * u] = live != 0.f ? s1 : 0.f;
        s[2 * u + 1] = live != 0.f ? s2 : 0.f;
      }
#pragma unroll
      for (int i = 0; i < 2 * LB_R; ++i) s[i] = wave_sum63(s[i]);
      if (lane == 63) *reinterpret_cast<float4*>(red[buf][wave]) = make_float4(s[0], s[1], s[2], s[3]);
      __syncthreads();
      float m[2 * LB_R] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float4 v = *reinterpret_cast<const float4*>(red[buf][w]);
        m[0] += v.x; m[1] += v.y; m[2] += v.z; m[3] += v.w;
      }
      buf ^= 1;
#pragma unroll
      for (int u = 0; u < LB_R; ++u) {
        if (on && q + u < pend) {
          const float m1 = m[2 * u] * invF, m2 = m[2 * u + 1] * invF;
          float x[VEC], o[VEC];
          Vec<E>::unpack(cur.h[u], x);
#pragma unroll
          for (int j = 0; j < VEC; ++j) {
            const float n = (x[j] - cur.st[u].x) * cur.st[u].y;
            o[j] = cur.st[u].y * (dn[u][j] - m1 - n * m2);
          }
          const uint4 ov = Vec<E>::pack(o);
          *reinterpret_cast<uint4*>(dh + (int64_t)(q + u) * F + c) = ov;
          Vec<E>::unpack(ov, o);
#pragma unroll
          for (int j = 0; j < VEC; ++j) ad[j] += o[j];
        }
      }
      cur = nxt;
    }
    if (on) {
      if (r == ebeg && pend == eend) {
        *reinterpret_cast<uint4*>(dgamma + (int64_t)e * F + c) = Vec<E>::pack(ag);
        *reinterpret_cast<uint4*>(dbeta + (int64_t)e * F + c) = Vec<E>::pack(ab);
        *reinterpret_cast<uint4*>(db + (int64_t)e * F + c) = Vec<E>::pack(ad);
      } else {
        float* p = part + (int64_t)(r == r0 ? lb_first_slot(blk) : lb_last_slot(nb, N, blk, e)) * 3 * F + c;
#pragma unroll
        for (int j = 0; j < VEC; j += 4) {
          *reinterpret_cast<float4*>(p + j) = make_float4(ag[j], ag[j + 1], ag[j + 2], ag[j + 3]);
          *reinterpret_cast<float4*>(p + F + j) = make_float4(ab[j], ab[j + 1], ab[j + 2], ab[j + 3]);
          *reinterpret_cast<float4*>(p + 2 * F + j) = make_float4(ad[j], ad[j + 1], ad[j + 2], ad[j + 3]);
        }
      }
    }
    r = pend;
  }
}

// The experts whose rows ln_bwd_kernel's blocks split: their pieces added in row order.
// Block (x, e): 256 threads take 1024 of the 3 F sums of expert e.
template <typename E>
__global__ void __launch_bounds__(256)
ln_bwd_reduce_kernel(const int32_t* offsets, int N, int F, int nb, const float* part, E* dgamma, E* dbeta, E* db) {
  const int e = blockIdx.y;
  const int ebeg = offsets[e], eend = offsets[e + 1];
  if (ebeg == eend) return;
  const int P = offsets[N];
  const int per = (P + nb - 1) / nb;
  const int b0 = ebeg / per, b1 = (eend - 1) / per;
  if (b0 == b1) return;
  const int q = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;
  if (q >= 3 * F) return;
  float4 s = *reinterpret_cast<const float4*>(
      part + (int64_t)(ebeg == b0 * per ? lb_first_slot(b0) : lb_last_slot(nb, N, b0, e)) * 3 * F + q);
  for (int b = b0 + 1; b <= b1; ++b) {
    const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)lb_first_slot(b) * 3 * F + q);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  E* out = (q < F ? dgamma : q < 2 * F ? dbeta : db) + (int64_t)e * F + q % F;   // F is a multiple of 64
  out[0] = cvt<E>(s.x); out[1] = cvt<E>(s.y); out[2] = cvt<E>(s.z); out[3] = cvt<E>(s.w);
}

template <typename E>
static void ln_bwd_fused(const Shape& s, const int32_t* offsets, const E* h, const float* stats, const E* g, const E* b,
                         const E* da, E* dh, E* dg, E* dbe, E* db, float* part, hipStream_t st) {
  const int N = (int)s.N, F = (int)s.H, nt = lb_threads(F / Vec<E>::N);
  const int nb = (int)workspace_layout(s).ln_blocks;
  auto go = [&](auto ACTc, auto NTc) {
    constexpr int ACT = decltype(ACTc)::value, NT = decltype(NTc)::value;
    DMOE_LAUNCH_NAMED("ln_bwd_kernel", (ln_bwd_kernel<E, ACT, NT>), dim3(nb), dim3(NT), 0, st, h, stats, offsets, N, F, g,
                      b, da, dh, dg, dbe, db, part);
  };
  auto nts = [&](auto ACTc) {
    if (nt == 64) go(ACTc, std::integral_constant<int, 64>{});
    else if (nt == 128) go(ACTc, std::integral_constant<int, 128>{});
    else if (nt == 256) go(ACTc, std::integral_constant<int, 256>{});
    else go(ACTc, std::integral_constant<int, 512>{});
  };
  if (s.act == DMOE_RELU) nts(std::integral_constant<int, DMOE_RELU>{});
  else nts(std::integral_constant<int, DMOE_GELU>{});
  DMOE_LAUNCH_NAMED("ln_bwd_reduce_kernel", ln_bwd_reduce_kernel<E>, dim3((unsigned)((3 * F + 1023) / 1024), (unsigned)N),
                    dim3(256), 0, st, offsets, N, F, nb, part, dg, dbe, db);
}

// chunks per lane for a row of F values: the smallest of 1, 2, 4, 8 that holds it
template <typename E> static int ln_chunks(int64_t F) {
  const int64_t per = (F / Vec<E>::N + 63) / 64;
  return per <= 1 ? 1 : per <= 2 ? 2 : per <= 4 ? 4 : 8;
}
template <typename E> static bool ln_width_ok(int64_t F) {
  return F % Vec<E>::N == 0 && F / Vec<E>::N <= 64 * LN_CHMAX;
}

static int ln_grid(const Shape& s) {
  const int64_t waves = std::max<int64_t>(1, std::min<int64_t>(s.P, 4096));
  return (int)((waves + LN_NT / 64 - 1) / (LN_NT / 64));
}

template <typename E, int ACT>
static void ln_fwd_act(const Shape& s, const int32_t* offsets, const E* h, const E* g, const E* b, E* a,
                       float* stats, hipStream_t st) {
  const int N = (int)s.N, F = (int)s.H, grid = ln_grid(s);
  switch (ln_chunks<E>(F)) {
    case 1: DMOE_LAUNCH((ln_act_fwd_kernel<E, 1, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, offsets, N, F, g, b, a, stats); break;
    case 2: DMOE_LAUNCH((ln_act_fwd_kernel<E, 2, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, offsets, N, F, g, b, a, stats); break;
    case 4: DMOE_LAUNCH((ln_act_fwd_kernel<E, 4, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, offsets, N, F, g, b, a, stats); break;
    default: DMOE_LAUNCH((ln_act_fwd_kernel<E, 8, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, offsets, N, F, g, b, a, stats); break;
  }
}
template <typename E>
static void ln_fwd(const Shape& s, const int32_t* offsets, const E* h, const E* g, const E* b, E* a,
                   float* stats, hipStream_t st) {
  if (s.act == DMOE_RELU) ln_fwd_act<E, DMOE_RELU>(s, offsets, h, g, b, a, stats, st);
  else ln_fwd_act<E, DMOE_GELU>(s, offsets, h, g, b, a, stats, st);
}

// scale and shift gradients first (they read da), then dh (which may overwrite da)
template <typename E, int ACT>
static void ln_bwd_act(const Shape& s, const int32_t* offsets, const E* h, const float* stats, const E* g,
                       const E* b, const E* da, E* dh, E* dg, E* db, hipStream_t st) {
  const int N = (int)s.N, F = (int)s.H, grid = ln_grid(s);
  with_lanes(colsum_lanes<E>(s, F), [&](auto CLc) {
    constexpr int CL = decltype(CLc)::value;
    DMOE_LAUNCH((ln_act_bwd_params_kernel<E, ACT, CL>), dim3((unsigned)colsum_blocks<E>(F, CL), (unsigned)N), dim3(CS_NT), 0,
                st, h, stats, offsets, F, g, b, da, dg, db);
  });
  switch (ln_chunks<E>(F)) {
    case 1: DMOE_LAUNCH((ln_act_bwd_rows_kernel<E, 1, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, stats, offsets, N, F, g, b, da, dh); break;
    case 2: DMOE_LAUNCH((ln_act_bwd_rows_kernel<E, 2, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, stats, offsets, N, F, g, b, da, dh); break;
    case 4: DMOE_LAUNCH((ln_act_bwd_rows_kernel<E, 4, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, stats, offsets, N, F, g, b, da, dh); break;
    default: DMOE_LAUNCH((ln_act_bwd_rows_kernel<E, 8, ACT>), dim3(grid), dim3(LN_NT), 0, st, h, stats, offsets, N, F, g, b, da, dh); break;
  }
}
template <typename E>
static void ln_bwd(const Shape& s, const int32_t* offsets, const E* h, const float* stats, const E* g, const E* b,
                   const E* da, E* dh, E* dg, E* db, hipStream_t st) {
  if (s.act == DMOE_RELU) ln_bwd_act<E, DMOE_RELU>(s, offsets, h, stats, g, b, da, dh, dg, db, st);
  else ln_bwd_act<E, DMOE_GELU>(s, offsets, h, stats, g, b, da, dh, dg, db, st);
}

// ---------------------------------------------------------------- linear layers
// Row-major operands: a layer's weight W [N, n_out, n_in], rows grouped by expert.

// Tile shape of an fp32 layer's row-grouped GEMMs (bf16 ones are picked per GEMM).
template <typename F> static void with_f32_tile(const Shape& s, F&& f) {
  if (use_fat_f32(s)) f(CfgF32{});
  else f(CfgF32Skinny{});
}
// the tile plan of a pass: heights for the F columns (a) and the D columns (b)
template <typename E>
static void block_plan(const Shape& s, const int32_t* offsets, const Plan& pl, hipStream_t st) {
  if constexpr (sizeof(E) == 2) {
    run_tile_plan(s, offsets, row_tile_rows(s, s.H), row_tile_rows(s, s.D), pl, st);
  } else {
    with_f32_tile(s, [&](auto cfg) { run_tile_plan(s, offsets, decltype(cfg)::TMR, decltype(cfg)::TMR, pl, st); });
  }
}
template <bool BT, int EPI, typename E>
static void lin_rows(const Shape& s, GemmArgs<E> p, hipStream_t st) {
  if constexpr (sizeof(E) == 2) {
    run_gemm2_rows<BT, EPI>(s, p, st);
  } else {
    with_f32_tile(s, [&](auto cfg) {
      using C = decltype(cfg);
      const int64_t mt_ub = (s.P + C::TMR - 1) / C::TMR + std::min<int64_t>(s.N, s.P);
      p.tscale = (p.N + C::BN - 1) / C::BN;
      run_gemm_f32<GROUP_M, false, BT, EPI, C>(p, mt_ub * p.tscale, st);
    });
  }
}

// C[rows, n_out] = A[rows, n_in] W_e^T + b_e
template <typename E>
static void lin_fwd(const Shape& s, const int32_t* offsets, const int32_t* tpre, const E* A, int n_in,
                    const E* W, const E* b, int n_out, E* Cp, hipStream_t st) {
  GemmArgs<E> p = args_m<E>(offsets, tpre, 0, (int)s.N);
  p.A = A; p.lda = n_in;
  p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
  p.C = Cp; p.ldc = n_out;
  p.bias = b; p.bias_gstride = n_out;
  p.N = n_out; p.K = n_in; p.act = s.act;
  lin_rows<false, EPI_BIAS>(s, p, st);
}

// dA[rows, n_in] = dC[rows, n_out] W_e   (W_e read as (n = input feature, k = output feature))
template <typename E>
static void lin_dgrad(const Shape& s, const int32_t* offsets, const int32_t* tpre, const E* dC, int n_out,
                      const E* W, int n_in, E* dA, hipStream_t st) {
  GemmArgs<E> p = args_m<E>(offsets, tpre, 0, (int)s.N);
  p.A = dC; p.lda = n_out;
  p.B = W; p.ldb = n_in; p.b_gstride = (int64_t)n_out * n_in;
  p.C = dA; p.ldc = n_in;
  p.N = n_in; p.K = n_out; p.act = s.act;
  lin_rows<true, EPI_STORE>(s, p, st);
}

// dW_e[n_out, n_in] = dC_e^T A_e over the expert's rows
template <typename E, typename CW>
static void lin_wgrad(const Shape& s, const int32_t* offsets, const int32_t* tact, const E* dC, int n_out,
                      const E* A, int n_in, E* dW, hipStream_t st) {
  const int64_t active_ub = std::min<int64_t>(s.N, s.P);
  const int mt = (n_out + CW::BM - 1) / CW::BM, nt = (n_in + CW::BN - 1) / CW::BN;
  GemmArgs<E> p = args_m<E>(offsets, tact, mt * nt, (int)s.N);
  p.A = dC; p.lda = n_out;
  p.B = A; p.ldb = n_in;
  p.C = dW; p.ldc = n_in; p.c_gstride = (int64_t)n_out * n_in;
  p.M = n_out; p.N = n_in; p.act = s.act;
  if constexpr (sizeof(E) == 2)
    run_gemm2<GROUP_K, true, true, EPI_STORE, CW::BM, CW::BN, CW::WM, CW::WN, CW::ST, CW::BK, CW::STO>(p, active_ub * mt * nt, st);
  else
    run_gemm_f32<GROUP_K, true, true, EPI_STORE, CW>(p, active_ub * mt * nt, st);
}

template <typename E>
static void colsum(const Shape& s, const int32_t* offsets, const E* X, int ncols, E* out, hipStream_t st) {
  run_colsum<E>(s, offsets, X, ncols, out, (const E*)nullptr, 0, (E*)nullptr, 0.f, st);
}

template <typename E> struct BlockP {
  const E *W1, *b1, *g1, *be1, *W2, *b2, *g2, *be2, *W3, *b3;
};
template <typename E> struct BlockG {
  E *W1, *b1, *g1, *be1, *W2, *b2, *g2, *be2, *W3, *b3;
};
template <typename E> struct BlockA {
  E *h1, *a1, *h2, *a2;
  float *st1, *st2;
};

template <typename E>
static void block_fwd(const Shape& s, const int32_t* offsets, const E* xp, const BlockP<E>& q, const BlockA<E>& t,
                      E* yp, const Plan& pl, hipStream_t st) {
  const int D = (int)s.D, F = (int)s.H;
  block_plan<E>(s, offsets, pl, st);
  lin_fwd<E>(s, offsets, pl.a, xp, D, q.W1, q.b1, F, t.h1, st);
  ln_fwd<E>(s, offsets, t.h1, q.g1, q.be1, t.a1, t.st1, st);
  lin_fwd<E>(s, offsets, pl.a, t.a1, F, q.W2, q.b2, F, t.h2, st);
  ln_fwd<E>(s, offsets, t.h2, q.g2, q.be2, t.a2, t.st2, st);
  lin_fwd<E>(s, offsets, pl.b, t.a2, F, q.W3, q.b3, D, yp, st);
}

// g2 holds da2 then dh2, g1 holds da1 then dh1 (each normalisation backward in place).
template <typename E, typename CW>
static void block_bwd(const Shape& s, const int32_t* offsets, const E* xp, const BlockP<E>& q, const BlockA<E>& t,
                      const E* dyp, E* g1, E* g2, E* dxp, const BlockG<E>& d, const Plan& pl, float* part,
                      hipStream_t st) {
  const int D = (int)s.D, F = (int)s.H;
  const int32_t* tact = pl.act;
  block_plan<E>(s, offsets, pl, st);
  lin_wgrad<E, CW>(s, offsets, tact, dyp, D, t.a2, F, d.W3, st);     // dW3 = dy^T a2
  colsum<E>(s, offsets, dyp, D, d.b3, st);                            // db3
  lin_dgrad<E>(s, offsets, pl.a, dyp, D, q.W3, F, g2, st);            // da2 = dy W3
  ln_bwd_fused<E>(s, offsets, t.h2, t.st2, q.g2, q.be2, g2, g2, d.g2, d.be2, d.b2, part, st);   // dh2, dg2, dbe2, db2
  lin_wgrad<E, CW>(s, offsets, tact, g2, F, t.a1, F, d.W2, st);       // dW2 = dh2^T a1
  lin_dgrad<E>(s, offsets, pl.a, g2, F, q.W2, F, g1, st);             // da1 = dh2 W2
  ln_bwd_fused<E>(s, offsets, t.h1, t.st1, q.g1, q.be1, g1, g1, d.g1, d.be1, d.b1, part, st);   // dh1, dg1, dbe1, db1
  lin_wgrad<E, CW>(s, offsets, tact, g1, F, xp, D, d.W1, st);         // dW1 = dh1^T x
  lin_dgrad<E>(s, offsets, pl.b, g1, F, q.W1, D, dxp, st);            // dx_perm = dh1 W1
}

template <typename E> static BlockP<E> params_of(const dmoe_ffblock_params* p) {
  auto c = [](const void* v) { return reinterpret_cast<const E*>(v); };
  return {c(p->W1), c(p->b1), c(p->g1), c(p->be1), c(p->W2), c(p->b2), c(p->g2), c(p->be2), c(p->W3), c(p->b3)};
}
template <typename E> static BlockG<E> grads_of(const dmoe_ffblock_params* p) {
  auto m = [](void* v) { return reinterpret_cast<E*>(v); };
  return {m(p->W1), m(p->b1), m(p->g1), m(p->be1), m(p->W2), m(p->b2), m(p->g2), m(p->be2), m(p->W3), m(p->b3)};
}
template <typename E> static BlockA<E> acts_of(const dmoe_ffblock_acts* a) {
  auto m = [](void* v) { return reinterpret_cast<E*>(v); };
  return {m(a->h1), m(a->a1), m(a->h2), m(a->a2), a->st1, a->st2};
}

static bool params_ok(const dmoe_ffblock_params* p) {
  if (!p) return false;
  for (const void* v : {p->W1, p->b1, p->g1, p->be1, p->W2, p->b2, p->g2, p->be2, p->W3, p->b3})
    if (!v) return false;
  return true;
}
static bool params_aligned(const dmoe_ffblock_params* p) {
  for (const void* v : {p->W1, p->b1, p->g1, p->be1, p->W2, p->b2, p->g2, p->be2, p->W3, p->b3})
    if (!aligned16(v)) return false;
  return true;
}
static bool acts_ok(const dmoe_ffblock_acts* a) {
  return a && a->h1 && a->a1 && a->st1 && a->h2 && a->a2 && a->st2;
}
static bool acts_aligned(const dmoe_ffblock_acts* a) {
  for (const void* v : {a->h1, a->a1, (void*)a->st1, a->h2, a->a2, (void*)a->st2})
    if (!aligned16(v)) return false;
  return true;
}
static bool ln_width_supported(const Shape& s) {
  return s.dtype == DMOE_BF16 ? ln_width_ok<bf16>(s.H) : ln_width_ok<float>(s.H);
}

}  // namespace dmoe

using namespace dmoe;

extern "C" int dmoe_ln_act_fwd(const dmoe_dims* dims, const int32_t* offsets, const void* h, const void* gamma,
                               const void* beta, void* a, float* stats, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !h || !gamma || !beta || !a || !stats) return DMOE_EINVAL;
  if (!ln_width_supported(s)) return DMOE_EUNSUPPORTED;
  for (const void* q : {h, gamma, beta, (const void*)a, (const void*)stats})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16)
    ln_fwd<bf16>(s, offsets, reinterpret_cast<const bf16*>(h), reinterpret_cast<const bf16*>(gamma),
                 reinterpret_cast<const bf16*>(beta), reinterpret_cast<bf16*>(a), stats, st);
  else
    ln_fwd<float>(s, offsets, reinterpret_cast<const float*>(h), reinterpret_cast<const float*>(gamma),
                  reinterpret_cast<const float*>(beta), reinterpret_cast<float*>(a), stats, st);
  return launch_status();
}

extern "C" int dmoe_ln_act_bwd(const dmoe_dims* dims, const int32_t* offsets, const void* h, const float* stats,
                               const void* gamma, const void* beta, const void* da, void* dh, void* dgamma,
                               void* dbeta, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !h || !stats || !gamma || !beta || !da || !dh || !dgamma || !dbeta) return DMOE_EINVAL;
  if (!ln_width_supported(s)) return DMOE_EUNSUPPORTED;
  for (const void* q : {h, (const void*)stats, gamma, beta, da, (const void*)dh, (const void*)dgamma,
                        (const void*)dbeta})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    ln_bwd<bf16>(s, offsets, c(h), stats, c(gamma), c(beta), c(da), m(dh), m(dgamma), m(dbeta), st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    ln_bwd<float>(s, offsets, c(h), stats, c(gamma), c(beta), c(da), m(dh), m(dgamma), m(dbeta), st);
  }
  return launch_status();
}

extern "C" int dmoe_expert_ffblock_fwd(const dmoe_dims* dims, const int32_t* offsets, const void* x_perm,
                                       const dmoe_ffblock_params* params, const dmoe_ffblock_acts* acts,
                                       void* y_perm, void* ws, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !params_ok(params) || !acts_ok(acts) || !y_perm || !ws) return DMOE_EINVAL;
  if (!ln_width_supported(s)) return DMOE_EUNSUPPORTED;
  if (!aligned16(x_perm) || !aligned16(y_perm) || !aligned16(ws) || !params_aligned(params) || !acts_aligned(acts))
    return DMOE_EUNSUPPORTED;
  const Plan pl =
      plan_at(reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + workspace_layout(s).tiles_off), s.N, true);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16) {
    const bf16* xp = reinterpret_cast<const bf16*>(x_perm);
    bf16* yp = reinterpret_cast<bf16*>(y_perm);
    block_fwd<bf16>(s, offsets, xp, params_of<bf16>(params), acts_of<bf16>(acts), yp, pl, st);
  } else {
    const float* xp = reinterpret_cast<const float*>(x_perm);
    float* yp = reinterpret_cast<float*>(y_perm);
    block_fwd<float>(s, offsets, xp, params_of<float>(params), acts_of<float>(acts), yp, pl, st);
  }
  return launch_status();
}

extern "C" int dmoe_expert_ffblock_bwd(const dmoe_dims* dims, const int32_t* offsets, const void* x_perm,
                                       const dmoe_ffblock_params* params, const dmoe_ffblock_acts* acts,
                                       const void* dy_perm, void* g1, void* g2, void* dx_perm,
                                       const dmoe_ffblock_params* grads, void* ws, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!offsets || !x_perm || !params_ok(params) || !acts_ok(acts) || !dy_perm || !g1 || !g2 || !dx_perm ||
      !params_ok(grads) || !ws)
    return DMOE_EINVAL;
  if (!ln_width_supported(s)) return DMOE_EUNSUPPORTED;
  for (const void* q : {x_perm, dy_perm, (const void*)g1, (const void*)g2, (const void*)dx_perm, (const void*)ws})
    if (!aligned16(q)) return DMOE_EUNSUPPORTED;
  if (!params_aligned(params) || !params_aligned(grads) || !acts_aligned(acts)) return DMOE_EUNSUPPORTED;
  const Plan pl =
      plan_at(reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + workspace_layout(s).tiles_off), s.N, true);
  float* part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(ws) + workspace_layout(s).ln_off);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.dtype == DMOE_BF16) {
    auto c = [](const void* q) { return reinterpret_cast<const bf16*>(q); };
    auto m = [](void* q) { return reinterpret_cast<bf16*>(q); };
    if (deep_wgrad(s))
      block_bwd<bf16, G2DW>(s, offsets, c(x_perm), params_of<bf16>(params), acts_of<bf16>(acts), c(dy_perm),
                            m(g1), m(g2), m(dx_perm), grads_of<bf16>(grads), pl, part, st);
    else
      block_bwd<bf16, G2DWShort>(s, offsets, c(x_perm), params_of<bf16>(params), acts_of<bf16>(acts), c(dy_perm),
                                 m(g1), m(g2), m(dx_perm), grads_of<bf16>(grads), pl, part, st);
  } else {
    auto c = [](const void* q) { return reinterpret_cast<const float*>(q); };
    auto m = [](void* q) { return reinterpret_cast<float*>(q); };
    if (use_fat_f32(s))
      block_bwd<float, CfgF32DW>(s, offsets, c(x_perm), params_of<float>(params), acts_of<float>(acts), c(dy_perm),
                                 m(g1), m(g2), m(dx_perm), grads_of<float>(grads), pl, part, st);
    else
      block_bwd<float, CfgF32>(s, offsets, c(x_perm), params_of<float>(params), acts_of<float>(acts), c(dy_perm),
                               m(g1), m(g2), m(dx_perm), grads_of<float>(grads), pl, part, st);
  }
  return launch_status();
}
