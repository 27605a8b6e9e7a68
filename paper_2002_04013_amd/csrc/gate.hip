// Structured gate, exact TopK over the expert grid and Eq. 1 weights
// (Sec. 3.2, Eq. 1, App. C), plus the gate's backward pass.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "gemm2.hpp"
#include "gemm_f32.hpp"

namespace dmoe {

struct GateArgs {
  const void* x; const void* Wg; const void* bg; const uint8_t* alive;
  int32_t* idx; float* w; float* g; float* scores;
  int T, D, d, M, k, dM, N;
};

// One token's certified selection by one lane, from its MFMA scores s64[d*M] (Sec. 3.2,
// Eq. 1, App. C):
//  * decision scores are the fp32 roundings of the scores;
//  * per dimension, the best min(K1, M) indices by (score desc, index asc), kept in
//    registers by an insertion network (ties keep the earlier, lower index);
//  * the cells whose rank product is at most K1 (the only cells that can be among
//    the K1 best: a cell with per-dimension ranks r_i is beaten by the
//    prod(r_i + 1) - 1 cells taking an equal or better index in every dimension),
//    ranked by their fp64 total of d fp32 values in dimension order, ties to the
//    lower flat index;
//  * K1 = k+1 cells (k if k = N) are ranked, and the selection is kept only if their
//    totals are separated by more than 2E, E = d (delta_max + amax 2^-23) with
//    delta = gam * ab[c] the bound on the score's accumulation error, and if the nonzero
//    scores are finite and span less than 2^25 in magnitude (beyond it an fp64 total of d
//    fp32 values may round and the dominance argument no longer holds exactly).  Returns
//    false (nothing written) otherwise.  A NaN score is below every other one;
//  * Eq. 1 weights over the chosen experts that are alive, from fp64 totals.
// CAP: list capacity, at least K1 (the callers pick 5 when K1 <= 5, else KMAX + 1;
// for ALIVE 7 when k <= 4, else KMAX + 3).
// EXACT: the scores are exact (ab is not read), E covers their rounding alone.
// ALIVE (TopK among the alive experts): the K1 = min(N, CAP) best cells are
// ranked the same way; walking them in order, the first k alive ones are the k best
// alive experts of the whole grid as soon as the k-th of them lies within those K1 (a
// cell outside the K1 best is beaten by all of them).  The selection is kept if the
// k-th alive cell is found there, the totals up to the cell after it are separated by
// more than 2E (or every cell was ranked), and the span condition holds; otherwise
// nothing is written (the token goes to the exact alive-first path).
// One lane per token is the form with the least work per token; the exact kernels below
// select with a wave per token, which has the lower latency.
template <int CAP, bool ALIVE, bool EXACT>
__device__ __forceinline__ bool select_token_cap(const double* s64, const float* ab, const uint8_t* alive, int d,
                                                 int M, int k, int N, float gam, int32_t* idx_out, float* w_out,
                                                 float* g_out) {
  const int K1 = ALIVE ? (N < CAP ? N : CAP) : (k < N ? k + 1 : k);
  const int L = K1 < M ? K1 : M;
  float lv[DMAX][CAP];
  int li[DMAX][CAP];
  float amax = 0.f, amin = 3.4e38f, dmax = 0.f;
#pragma unroll
  for (int i = 0; i < DMAX; ++i) {
#pragma unroll
    for (int p = 0; p < CAP; ++p) { lv[i][p] = -INFINITY; li[i][p] = 0; }
    if (i < d) {
      for (int u = 0; u < M; ++u) {
        float v = (float)s64[i * M + u];
        int id = u;
        const float av = fabsf(v);
        if (av > 0.f) { amax = fmaxf(amax, av); amin = fminf(amin, av); }
        if constexpr (!EXACT) dmax = fmaxf(dmax, gam * ab[i * M + u]);
#pragma unroll
        for (int p = 0; p < CAP; ++p) {
          const bool sw = v > lv[i][p];
          const float ov = lv[i][p];
          const int oi = li[i][p];
          lv[i][p] = sw ? v : ov; li[i][p] = sw ? id : oi;
          v = sw ? ov : v; id = sw ? oi : id;
        }
      }
    }
  }
  // top K1 cells: fp64 total, flat index, and the grid indices packed 8 bits per dim
  double tv[CAP];
  int tf[CAP], tu[CAP];
#pragma unroll
  for (int p = 0; p < CAP; ++p) { tv[p] = -INFINITY; tf[p] = 0x7fffffff; tu[p] = 0; }
  auto insert = [&](double v, int f, int uu) {
#pragma unroll
    for (int p = 0; p < CAP; ++p) {
      const bool sw = v > tv[p] || (v == tv[p] && f < tf[p]);
      const double ov = tv[p];
      const int of = tf[p], ou = tu[p];
      tv[p] = sw ? v : ov; tf[p] = sw ? f : of; tu[p] = sw ? uu : ou;
      v = sw ? ov : v; f = sw ? of : f; uu = sw ? ou : uu;
    }
  };
  // span 2^25; infinite scores (their totals may be NaN, which the lists cannot hold) are
  // left to the exact path whatever the others are
  if (!(amax < INFINITY) || (amax > 0.f && !(amax <= amin * 33554432.f))) return false;
  {
    // odometer over the rank digits r_0 .. r_{d-1} (last digit fastest), visiting only
    // the tuples with prod(r_i + 1) <= K1: a digit whose prefix product would exceed
    // K1 carries into the previous digit at once
    int r[DMAX];
#pragma unroll
    for (int i = 0; i < DMAX; ++i) r[i] = 0;
    for (int guard = 0; guard < 4096; ++guard) {
      int prod = 1;
#pragma unroll
      for (int i = 0; i < DMAX; ++i) if (i < d) prod *= r[i] + 1;
      if (prod <= K1) {
        double tot = 0.0;
        int flat = 0, uu = 0;
#pragma unroll
        for (int i = 0; i < DMAX; ++i) {
          if (i < d) {
            // element r[i] of the lists, by selects (the lists stay in registers)
            float pv = lv[i][0];
            int pi = li[i][0];
#pragma unroll
            for (int p = 1; p < CAP; ++p) { pv = r[i] == p ? lv[i][p] : pv; pi = r[i] == p ? li[i][p] : pi; }
            tot += (double)pv;
            flat = flat * M + pi;
            uu |= pi << (8 * i);
          }
        }
        insert(tot, flat, uu);
      }
      // next tuple: bump the last digit; a digit that reaches L, or makes the product
      // exceed K1 (so every larger value of it does too), resets and carries
      bool carry = true;
#pragma unroll
      for (int i = DMAX - 1; i >= 0; --i) {
        if (i < d && carry) {
          r[i] += 1;
          int pr = 1;
#pragma unroll
          for (int ii = 0; ii < DMAX; ++ii) if (ii < d) pr *= r[ii] + 1;
          if (r[i] >= L || pr > K1) r[i] = 0;
          else carry = false;
        }
      }
      if (carry) break;                  // every digit wrapped: done
    }
  }
  if constexpr (ALIVE) {
    // the first k alive cells among the K1 best; position of the k-th
    int pk = -1, cnt = 0;
#pragma unroll
    for (int p = 0; p < CAP; ++p) {
      const bool live = p < K1 && cnt < k && (alive == nullptr || alive[tf[p]] != 0);
      if (live) {
        ++cnt;
        if (cnt == k) pk = p;
      }
    }
    if (pk < 0) return false;
    if (pk + 1 >= K1 && K1 < N) return false;      // the cell after the k-th is not ranked
    const double E = (double)d * ((double)dmax + (double)amax * 1.1920928955078125e-7);
    bool sep = true;
#pragma unroll
    for (int j = 0; j + 1 < CAP; ++j)
      if (j <= pk && j + 1 < K1) sep = sep && (tv[j] - tv[j + 1] > 2.0 * E);
    if (!sep) return false;
    // keep only the alive cells, in order: compact positions 0 .. pk
    int w = 0;
#pragma unroll
    for (int p = 0; p < CAP; ++p) {
      if (p <= pk && (alive == nullptr || alive[tf[p]] != 0)) {
        // move entry p to slot w (w <= p): selects over the register arrays
        const double vv = tv[p];
        const int ff = tf[p], uu = tu[p];
#pragma unroll
        for (int q = 0; q < CAP; ++q)
          if (q == w) { tv[q] = vv; tf[q] = ff; tu[q] = uu; }
        ++w;
      }
    }
  } else {
    const double E = (double)d * ((double)dmax + (double)amax * 1.1920928955078125e-7);
    bool sep = true;
#pragma unroll
    for (int j = 0; j + 1 < CAP; ++j)
      if (j + 1 < K1) sep = sep && (tv[j] - tv[j + 1] > 2.0 * E);
    if (!sep) return false;
  }
  // Eq. 1 weights from the fp64 totals of the chosen experts, over the alive ones
  constexpr int KJ = CAP < KMAX ? CAP : KMAX;      // k <= K1 <= CAP
  double gx[KJ];
  bool live[KJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) live[j] = j < k && (alive == nullptr || alive[tf[j]] != 0);
  double m = -1.0e308;
  bool any = false;
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    gx[j] = 0.0;
    if (j < k) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < DMAX; ++i) if (i < d) t += s64[i * M + ((tu[j] >> (8 * i)) & 0xff)];
      gx[j] = t;
      if (live[j]) { any = true; m = t > m ? t : m; }
    }
  }
  float ex[KJ];
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    ex[j] = live[j] ? expf((float)(gx[j] - m)) : 0.f;
    sum += ex[j];
  }
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    if (j < k) {
      idx_out[j] = tf[j];
      w_out[j] = any ? ex[j] / sum : 0.f;
      if (g_out) g_out[j] = (float)gx[j];
    }
  }
  return true;
}

template <bool ALIVE, bool EXACT = false>
__device__ __forceinline__ bool select_token(const double* s64, const float* ab, const uint8_t* alive, int d, int M,
                                             int k, int N, float gam, int32_t* idx_out, float* w_out, float* g_out) {
  if constexpr (ALIVE) {      // k + 3 cells ranked: up to two dead ones ahead of the k-th alive
    if (k <= 4) return select_token_cap<7, true, EXACT>(s64, ab, alive, d, M, k, N, gam, idx_out, w_out, g_out);
    return select_token_cap<KMAX + 3, true, EXACT>(s64, ab, alive, d, M, k, N, gam, idx_out, w_out, g_out);
  }
  if (k + 1 <= 5) return select_token_cap<5, false, EXACT>(s64, ab, alive, d, M, k, N, gam, idx_out, w_out, g_out);
  return select_token_cap<KMAX + 1, false, EXACT>(s64, ab, alive, d, M, k, N, gam, idx_out, w_out, g_out);
}

// ---------------------------------------------------------------- bf16: MFMA scores + certificate
//
// Scores are computed on bf16 MFMA: products of bf16 values are exact in fp32, 32 of
// them are summed per MFMA chunk pair in fp32, and the chunk sums are added in fp64.
// A second MFMA over |x|.|w| gives A = sum_k |x_k w_k|, which bounds the accumulation
// error of each score:  |S - exact| <= delta = (gamma_32 + (D/32 + 8) 2^-52) A,
// gamma_n = n u / (1 - n u) with u = 2^-23 (no assumption about the MFMA's internal
// rounding beyond single-precision operations, directed rounding included).  Decision
// scores of the GPU and of an exact computation then differ by at most delta + 1 ulp
// each, a cell total by at most d (delta + ulp) =: E.  If the k+1 best cells (k when
// k = N) are separated by gaps larger than 2E, the exact scores give the same TopK in
// the same order; such tokens are certified.  The others are appended to a device
// queue and recomputed with exact fp64 accumulation by gate_exact_sparse_kernel.

constexpr int GM_TOK = 32;        // tokens per block (one MFMA row block)
constexpr int GM_RING = 2;        // x groups (32 tokens x 64 d_model, 4 KB) in flight per wave
// Waves per block (each a share of the d_model groups): 2 from d_model 2048 on, else 1.
// A 2-slot ring keeps a block's LDS small (8 KB per slot and wave with 32 gate columns),
// so that several blocks share a compute unit and one block's selection overlaps the
// others' loads.
constexpr int gm_kw(int64_t D) { return D >= 2048 ? 2 : 1; }
constexpr int GX_NT = 512;        // exact recomputation: threads per token

struct GateMfmaArgs {
  GateArgs a;
  float gam;                       // gamma_32 + (D/32+8) 2^-52, times 1/(1 - gamma_D)
  int32_t* queue;                  // [0] count, [GQ_HEAD + i] token ids
};

__device__ __forceinline__ void g2l16(const void* g, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 16, 0, 0);
}

// A block of KW waves scores 32 tokens against all d*M gate columns; wave w takes
// the d_model groups w, w + KW, ... (groups of 64 values).  x and Wg stream
// through a per-wave LDS ring of GM_RING groups (direct global->LDS loads, 8 rows x
// 128 bytes per instruction, 16-byte chunks XOR-swizzled by row): a slot holds 32
// token rows, then 32*CB gate-column rows.  Within a group, lane half h holds
// d_model offsets 32h .. 32h+31 and MFMA chunk j takes 32h+8j .. 32h+8j+7 from both
// operands (the contraction order is permuted identically for x and Wg).  The
// waves' fp64 partial sums are added in wave order in LDS, then one lane per token
// selects.
// ALIVE: TopK among the alive experts (the certified selection extended until k alive
// cells are decided; see select_token_cap).
template <int CB, int KW, bool ALIVE = false>   // 32-column blocks of the d*M gate columns; waves
__global__ void __launch_bounds__(64 * KW) gate_topk_mfma(GateMfmaArgs ga) {
  const GateArgs& a = ga.a;
  extern __shared__ __align__(1024) unsigned char sm[];
  constexpr int SLOT = 4096 * (1 + CB);          // bytes per ring slot
  constexpr int LPG = 4 * (1 + CB);              // load instructions per group
  const int dM = a.dM;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = blockIdx.x * GM_TOK;
  const bf16* x = reinterpret_cast<const bf16*>(a.x);
  const bf16* W = reinterpret_cast<const bf16*>(a.Wg);
  const bf16* bg = reinterpret_cast<const bf16*>(a.bg);
  const int tok = lane & 31, half = lane >> 5;
  const int NG = a.D / 64;
  const int ng = NG > wv ? (NG - wv + KW - 1) / KW : 0;         // groups of this wave
  char* ring = reinterpret_cast<char*>(sm) + wv * (GM_RING * SLOT);
  // instruction q fills rows 8q .. 8q+7 of the slot (q < 4: tokens, then gate columns);
  // lane -> row 8q + lane/8, chunk lane%8 stored at position (lane%8) ^ (row%8)
  const int lrow = lane >> 3, lch = lane & 7;
  auto issue = [&](int m) {                       // the wave's m-th group
    char* slot = ring + (m % GM_RING) * SLOT;
    const int64_t k0 = (int64_t)64 * (wv + KW * m);
#pragma unroll
    for (int q = 0; q < 4 * (1 + CB); ++q) {
      const int r = 8 * q + lrow;
      const int c = lch ^ (r & 7);
      const bf16* src;
      if (q < 4) src = x + (int64_t)min(t0 + r, a.T - 1) * a.D;
      else src = W + (int64_t)min(r - 32, dM - 1) * a.D;
      g2l16(src + k0 + 8 * c, slot + q * 1024);
    }
  };
  // fragment of slot row `row`, chunk 4*half + jj
  auto frag = [&](int m, int row, int jj) {
    const char* slot = ring + (m % GM_RING) * SLOT;
    const int c = (4 * half + jj) ^ (row & 7);
    return *reinterpret_cast<const bf16x8_t*>(slot + row * 128 + c * 16);
  };
#pragma unroll
  for (int m = 0; m < GM_RING; ++m)
    if (m < ng) issue(m);

  double acc[CB][16];
  f32x16_t aacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[cb][r] = 0.0; aacc[cb][r] = 0.f; }
  for (int m = 0; m < ng; ++m) {
    // Vector-memory operations retire in issue order, and group m is followed by the
    // groups issued after it, LPG loads each: once at most that many are
    // outstanding, group m has landed.
    static_assert(GM_RING == 2, "one group in flight behind the current one");
    if (m + 1 < ng) wait_vmcnt<LPG>(); else wait_vmcnt<0>();
    f32x16_t c[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) c[cb][r] = 0.f;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const bf16x8_t xq = frag(m, tok, jj);
      const uint4 xu = __builtin_bit_cast(uint4, xq);
      const uint4 xa = make_uint4(xu.x & 0x7fff7fffu, xu.y & 0x7fff7fffu, xu.z & 0x7fff7fffu, xu.w & 0x7fff7fffu);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const bf16x8_t wq = frag(m, 32 + 32 * cb + tok, jj);
        const uint4 wu = __builtin_bit_cast(uint4, wq);
        const uint4 wa = make_uint4(wu.x & 0x7fff7fffu, wu.y & 0x7fff7fffu, wu.z & 0x7fff7fffu, wu.w & 0x7fff7fffu);
        c[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wq, xq, c[cb], 0, 0, 0);
        aacc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wa),
                                                          __builtin_bit_cast(bf16x8_t, xa), aacc[cb], 0, 0, 0);
      }
      if (jj & 1) {                      // every 32 products the fp32 sums move to fp64
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int r = 0; r < 16; ++r) { acc[cb][r] += (double)c[cb][r]; c[cb][r] = 0.f; }
      }
    }
    // every lane has read group m from its slot (the wave's LDS reads retire in order
    // before the refill is issued); refill it with group m + RING
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), vmcnt/expcnt untouched
    asm volatile("" ::: "memory");
    if (m + GM_RING < ng) issue(m + GM_RING);
  }

  // partial sums to LDS in wave order (rows padded to an odd word count: distinct
  // banks per token), then one lane per token selects
  wait_vmcnt<0>();
  __syncthreads();                       // both rings drained before their memory is reused
  const int SLD = dM + 1;
  double* s64 = reinterpret_cast<double*>(sm);                 // [32][SLD]
  float* ab = reinterpret_cast<float*>(s64 + GM_TOK * SLD);    // [32][SLD]
  for (int w = 0; w < KW; ++w) {
    if (wv == w) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int cc = cb * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
          if (cc < dM) {
            if (w == 0) {
              s64[tok * SLD + cc] = acc[cb][r] + (bg ? (double)bf2f(bg[cc]) : 0.0);
              ab[tok * SLD + cc] = aacc[cb][r];
            } else {
              s64[tok * SLD + cc] += acc[cb][r];
              ab[tok * SLD + cc] += aacc[cb][r];
            }
          }
        }
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < GM_TOK && t0 + (int)threadIdx.x < a.T) {
    const int t = t0 + threadIdx.x;
    const bool ok = select_token<ALIVE>(s64 + lane * SLD, ab + lane * SLD, a.alive, a.d, a.M, a.k, a.N, ga.gam,
                                       a.idx + (int64_t)t * a.k, a.w + (int64_t)t * a.k,
                                       a.g ? a.g + (int64_t)t * a.k : nullptr);
    if (!ok) ga.queue[GQ_HEAD + atomicAdd(ga.queue, 1)] = t;
    if (ok && a.scores)
      for (int c = 0; c < dM; ++c) a.scores[(int64_t)t * dM + c] = (float)s64[lane * SLD + c];
  }
}

// Order-preserving 64-bit image of an fp64 value (larger value, larger key; no NaN).
__device__ __forceinline__ uint64_t ord64(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
// Cell keys (live, total, ~flat) compared lexicographically: alive first (when ranked
// that way), then the larger total, then the lower flat index (larger ~flat).
__device__ __forceinline__ bool cell_gt(uint32_t al, uint64_t at, uint32_t an, uint32_t bl, uint64_t bt,
                                        uint32_t bn) {
  return (al > bl) | ((al == bl) & ((at > bt) | ((at == bt) & (an > bn))));
}

// Element q (compile-time after unrolling) of a 16-byte vector, as a float.
template <typename E> __device__ __forceinline__ float vec_elem(const uint4& v, int q);
template <> __device__ __forceinline__ float vec_elem<float>(const uint4& v, int q) {
  return __uint_as_float(q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w);
}
template <> __device__ __forceinline__ float vec_elem<bf16>(const uint4& v, int q) {
  const uint32_t w = (q >> 1) == 0 ? v.x : (q >> 1) == 1 ? v.y : (q >> 1) == 2 ? v.z : v.w;
  return __uint_as_float((q & 1) ? (w & 0xffff0000u) : (w << 16));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t u64_max_dpp(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)v, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(v >> 32), (int)(uint32_t)(v >> 32), CTRL,
                                                            ROWS, 0xf, false);
  const uint64_t o = ((uint64_t)hi << 32) | lo;
  return o > v ? o : v;
}

// Maximum of a 64-bit value over the wave (every lane gets it): within each row of 16
// lanes by DPP exchanges (lane i with i^1, i^2, 7-i, 15-i), then row r-1's last lane into
// row r (rows 1 and 3) and lane 31 into rows 2 and 3, so that lane 63 holds the maximum.
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  v = u64_max_dpp<0xB1, 0xf>(v);       // quad_perm [1,0,3,2]
  v = u64_max_dpp<0x4E, 0xf>(v);       // quad_perm [2,3,0,1]
  v = u64_max_dpp<0x141, 0xf>(v);      // row_half_mirror
  v = u64_max_dpp<0x140, 0xf>(v);      // row_mirror
  v = u64_max_dpp<0x142, 0xa>(v);      // row_bcast:15
  v = u64_max_dpp<0x143, 0xc>(v);      // row_bcast:31
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
}

// The rank tuples (r_0 .. r_{d-1}) with prod(r_i + 1) <= K1, in order of the product: the
// cells of a grid that can be among its K1 best (a cell with per-dimension ranks r_i is
// beaten by the prod(r_i + 1) - 1 cells that take an equal or better index in every
// dimension).  Those of a smaller K1 are a prefix.  4 bits per digit.
constexpr int RANK_KMAX = KMAX + 3;      // largest K1
constexpr int RANK_TUPLES = 96;          // 93 tuples for d = 4, K1 = 11
struct RankTable {
  uint16_t tup[DMAX][RANK_TUPLES];
  uint8_t cnt[DMAX][RANK_KMAX + 1];
};
constexpr RankTable make_rank_table() {
  RankTable q{};
  for (int d = 1; d <= DMAX; ++d) {
    int n = 0;
    for (int prod = 1; prod <= RANK_KMAX; ++prod) {
      for (int r0 = 0; r0 < prod; ++r0)
        for (int r1 = 0; r1 < (d > 1 ? prod : 1); ++r1)
          for (int r2 = 0; r2 < (d > 2 ? prod : 1); ++r2)
            for (int r3 = 0; r3 < (d > 3 ? prod : 1); ++r3)
              if ((r0 + 1) * (r1 + 1) * (r2 + 1) * (r3 + 1) == prod)
                q.tup[d - 1][n++] = (uint16_t)(r0 | (r1 << 4) | (r2 << 8) | (r3 << 12));
      q.cnt[d - 1][prod] = (uint8_t)n;
    }
  }
  return q;
}
static __device__ const RankTable rank_table = make_rank_table();

// Orders the LDS operations of one wave for the compiler; the hardware keeps their order.
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// This lane's candidate tuples (the cells ranked for K1) and how many there are.
struct RankTuples { int cnt, tup[2]; };
template <bool ALIVE> __device__ __forceinline__ int rank_k1(const GateArgs& a) {
  return ALIVE ? min(a.N, RANK_KMAX) : a.k;
}
template <bool ALIVE> __device__ __forceinline__ RankTuples rank_tuples(const GateArgs& a) {
  const int lane = threadIdx.x & 63;
  RankTuples r;
  r.cnt = rank_table.cnt[a.d - 1][rank_k1<ALIVE>(a)];
  r.tup[0] = rank_table.tup[a.d - 1][lane];
  r.tup[1] = rank_table.tup[a.d - 1][min(lane + 64, RANK_TUPLES - 1)];
  return r;
}

// Per-wave LDS of the selection.
constexpr int RANK_LIVE = 1 << 30;       // N <= 16384
constexpr int DEC_ZERO = DM_MAX + 4 * DMAX;
struct SelectScratch {
  float dec[DEC_ZERO + 4];               // decision scores, each dimension padded to 4 with -inf; a 0
  float lv[DMAX][RANK_KMAX + 1];         // per dimension, the best indices: score and index
  int li[DMAX][RANK_KMAX + 1];
  double tot[RANK_TUPLES];               // candidate cells: total, flat index
  int flat[RANK_TUPLES];
  int rf[RANK_KMAX + 1], ru[RANK_KMAX + 1];   // by rank: flat index (bit 30: the expert responds), grid indices (8 bits each)
  int own[RANK_KMAX + 1];                     // by rank: the candidate that wrote it
};

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t u32_max_dpp(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
  return o > v ? o : v;
}
// As wave_max_u64, of 32 bits.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = u32_max_dpp<0xB1, 0xf>(v);
  v = u32_max_dpp<0x4E, 0xf>(v);
  v = u32_max_dpp<0x141, 0xf>(v);
  v = u32_max_dpp<0x140, 0xf>(v);
  v = u32_max_dpp<0x142, 0xa>(v);
  v = u32_max_dpp<0x143, 0xc>(v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// This lane takes the previous lane's value (lane 0 its own); the list below lies in a row of 16.
__device__ __forceinline__ uint32_t shift_up(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
}

// TopK by its definition for one token, by one wave, in one pass over every cell of the grid:
// lane l takes the cells l, l + 64, ... (mixed-radix digits advanced by 64 per cell), the
// totals adding the d decision scores in fp64 in dimension order, ranked (alive first when
// ALIVE, total desc, flat asc).  The k best so far lie in lanes 0 .. k - 1, best first; the
// few cells of a step that beat the k-th (a ballot) are inserted one by one, at their count of
// better entries; of the first 64 cells, most of which would be, the k best are taken by k rounds
// of a maximum (ranking them by counting is 64 steps, which the four waves of a SIMD share).  A
// step's alive flags are loaded RA_U steps at a time.
// Reached where a ranking of the likely cells does not decide: fewer than k alive among them,
// or totals that may round.  Bound by the latency of a step's and of an insertion's chain.  The
// gate call with a fifth of the experts alive, D = 512, fp32, as k rounds over every cell /
// with a sorted list of k cells in every lane / this form: T = 8192, 15625 experts, k = 8
// 3412 / 1072 / 381 us; 14641 experts, k = 4 1498 / 702 / 294 us; 4096 experts, k = 8
// 622 / 451 / 138 us.  T = 836, D = 1984, 256 experts, k = 6, 30% alive: 54 / 32 / 35 us (42 with
// the first cells ranked by counting).
constexpr int RA_U = 4;
template <bool ALIVE>
__device__ __forceinline__ void rank_all_wave(const GateArgs& a, const float* dec, int M4, int* rf, int* ru) {
  const int lane = threadIdx.x & 63;
  const int d = a.d, M = a.M, N = a.N, k = a.k;
  int u[DMAX], st[DMAX], at[DMAX];                                   // digits, their steps, the dimensions' scores
  {
    int rl = lane, rs = 64;
#pragma unroll
    for (int i = DMAX - 1; i >= 0; --i) {
      u[i] = 0; st[i] = 0; at[i] = DEC_ZERO;                         // dimensions past d add 0
      if (i < d) { u[i] = rl % M; rl /= M; st[i] = rs % M; rs /= M; at[i] = i * M4; }
    }
  }
  uint32_t el = 0u, en = 0u;                                         // this lane's entry: below every cell
  uint64_t et = 0ull;
  uint32_t kl = 0u, kn = 0u;                                         // the k-th entry
  uint64_t kt = 0ull;
  auto kth = [&]() {
    kl = (uint32_t)__builtin_amdgcn_readlane((int)el, k - 1);
    kn = (uint32_t)__builtin_amdgcn_readlane((int)en, k - 1);
    kt = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(et >> 32), k - 1) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)et, k - 1);
  };
  for (int f0 = 0; f0 < N; f0 += 64 * RA_U) {
    uint32_t live[RA_U];
    uint64_t tt[RA_U];
#pragma unroll
    for (int q = 0; q < RA_U; ++q) {
      live[q] = 1u;
      if (ALIVE && a.alive != nullptr) live[q] = a.alive[min(f0 + 64 * q + lane, N - 1)];
    }
#pragma unroll
    for (int q = 0; q < RA_U; ++q) {
      double tot = 0.0;
      int carry = 0;
#pragma unroll
      for (int i = 0; i < DMAX; ++i) tot += (double)dec[at[i] + u[i]];   // digits stay in [0, M)
      tt[q] = ord64(tot == tot ? tot + 0.0 : -INFINITY);             // -0 and +0 are one value
#pragma unroll
      for (int i = DMAX - 1; i >= 0; --i) {                          // digits of f + 64
        u[i] += st[i] + carry;
        carry = u[i] >= M;
        u[i] -= carry ? M : 0;
      }
    }
#pragma unroll
    for (int q = 0; q < RA_U; ++q) {
      const int f = f0 + 64 * q + lane;
      const uint32_t n = ~(uint32_t)f, l = live[q] != 0u ? 1u : 0u;
      auto take = [&](int s, uint32_t& cl, uint64_t& ct, uint32_t& cn) {     // the cell of lane s
        cl = (uint32_t)__builtin_amdgcn_readlane((int)l, s);
        cn = (uint32_t)__builtin_amdgcn_readlane((int)n, s);
        ct = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(tt[q] >> 32), s) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tt[q], s);
      };
      if (q == 0 && f0 == 0) {                                       // the first cells: k rounds of a maximum
        bool in = f < N;
        for (int j = 0; j < min(N, k); ++j) {
          const bool alive = __ballot(in && l != 0u) != 0ull;
          const bool cand = in && (!alive || l != 0u);
          const uint64_t best = wave_max_u64(cand ? tt[q] : 0ull);   // no image is 0
          const int s = __builtin_ctzll(__ballot(cand && tt[q] == best));
          if (lane == j) { el = alive ? 1u : 0u; et = best; en = ~(uint32_t)s; }
          in = in && lane != s;
        }
        kth();
        continue;
      }
      uint64_t in = __ballot(f < N && cell_gt(l, tt[q], n, kl, kt, kn));
      while (in) {
        const int s = __builtin_ctzll(in);
        in &= in - 1;
        uint32_t cl, cn;
        uint64_t ct;
        take(s, cl, ct, cn);
        if (!cell_gt(cl, ct, cn, kl, kt, kn)) continue;              // a cell of this step took its place
        const int pos = __popcll(__ballot(lane < k && cell_gt(el, et, en, cl, ct, cn)));
        const uint32_t pl = shift_up(el), pn = shift_up(en);
        const uint64_t pt = ((uint64_t)shift_up((uint32_t)(et >> 32)) << 32) | shift_up((uint32_t)et);
        el = lane == pos ? cl : lane > pos ? pl : el;
        et = lane == pos ? ct : lane > pos ? pt : et;
        en = lane == pos ? cn : lane > pos ? pn : en;
        kth();
      }
    }
  }
  if (lane < k) {                                                    // k <= N: every entry is a cell
    const int f = (int)~en;
    int rem = f, uu = 0;
#pragma unroll
    for (int i = DMAX - 1; i >= 0; --i)
      if (i < d) { uu |= (rem % M) << (8 * i); rem /= M; }
    rf[lane] = f | (a.alive == nullptr || a.alive[f] != 0 ? RANK_LIVE : 0);
    ru[lane] = uu;
  }
  wave_lds_sync();
}

// One token's exact selection by one wave from its fp64 scores sc[d*M] in LDS: the same
// definition as select_token_cap without a certificate (the scores are exact).  Nothing is
// serial in k or M: a lane holds one or two gate columns and counts the columns of its
// dimension that beat it, which is the column's rank; a lane holds one or two candidate
// tuples and counts the candidates that beat its total.  Equal values are found by reading
// the rank slots back, and ranked again by (value desc, index asc).
// ALIVE: K1 = min(N, 11) cells are ranked and the first k alive ones taken; with
// fewer alive among them, or where fp64 totals may round (nonzero scores spanning more than
// 2^26), every cell of the grid is ranked.
template <bool ALIVE>
__device__ __forceinline__ void select_wave(const GateArgs& a, const RankTuples& rt, const double* sc,
                                            SelectScratch& q, int t) {
  const int lane = threadIdx.x & 63;
  const int d = a.d, M = a.M, k = a.k, N = a.N, dM = a.dM;
  const int M4 = (M + 3) & ~3;
  const int K1 = rank_k1<ALIVE>(a);
  const int L = min(K1, M);
  // decision scores (a NaN ranks with -inf, last), their span, and safe contents for the
  // rank slots
  int ci[2], cu[2];
  float cv[2];
  float amax = 0.f, amin = 3.4e38f;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = lane + 64 * h;
    ci[h] = (c >= M) + (c >= 2 * M) + (c >= 3 * M);
    cu[h] = c - ci[h] * M;
    cv[h] = 0.f;
    if (c < dM) {
      const float v = (float)sc[c], av = fabsf(v);
      cv[h] = v == v ? v : -INFINITY;
      q.dec[ci[h] * M4 + cu[h]] = cv[h];
      if (av > 0.f) { amax = fmaxf(amax, av); amin = fminf(amin, av); }
    }
  }
  if (lane == 0) q.dec[DEC_ZERO] = 0.f;
  for (int p = lane; p < d * (M4 - M); p += 64) q.dec[(p / (M4 - M)) * M4 + M + p % (M4 - M)] = -INFINITY;
  if (lane < DMAX * (RANK_KMAX + 1)) { (&q.lv[0][0])[lane] = -INFINITY; (&q.li[0][0])[lane] = 0; }
  if (lane <= RANK_KMAX) { q.rf[lane] = min(lane, N - 1); q.ru[lane] = 0; q.own[lane] = -1; }
  // magnitudes are not negative, so their bit patterns are ordered as they are
  amax = __uint_as_float(wave_max_u32(__float_as_uint(amax)));
  amin = __uint_as_float(~wave_max_u32(~__float_as_uint(amin)));
  bool full = amax > 0.f && !(amax <= amin * 67108864.f);            // span 2^26
  wave_lds_sync();
  // rank of each column in its dimension
  int rk[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    rk[h] = L;
    if (lane + 64 * h < dM) {
      const float* dv = q.dec + ci[h] * M4;
      int r = 0;
#pragma unroll 8
      for (int u = 0; u < M4; u += 4) {
        const float4 o = *reinterpret_cast<const float4*>(dv + u);
        r += (o.x > cv[h]) + (o.y > cv[h]) + (o.z > cv[h]) + (o.w > cv[h]);
      }
      rk[h] = r;
    }
  }
  auto put_lists = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (rk[h] < L) { q.lv[ci[h]][rk[h]] = cv[h]; q.li[ci[h]][rk[h]] = cu[h]; }
    wave_lds_sync();
  };
  put_lists();
  bool clash = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) clash |= rk[h] < L && q.li[ci[h]][rk[h]] != cu[h];
  if (__ballot(clash)) {                                             // equal scores: by index
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (rk[h] < L) {
        const float* dv = q.dec + ci[h] * M4;
        for (int u = 0; u < cu[h]; ++u) rk[h] += dv[u] == cv[h];
      }
    put_lists();
  }
  // candidate cells
  const int cnt = rt.cnt;
  double tv[2];
  int tf[2], tu[2];
  bool tk[2], lv[2] = {false, false};   // lv: alive, loaded while the ranks are counted
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int p = lane + 64 * h;
    tv[h] = -INFINITY; tf[h] = 0x7fffffff; tu[h] = 0; tk[h] = p < cnt;
    if (p < cnt) {
      const int tup = rt.tup[h];
      double tot = 0.0;
      int flat = 0, uu = 0;
#pragma unroll
      for (int i = 0; i < DMAX; ++i) {
        if (i < d) {
          const int r = (tup >> (4 * i)) & 15;
          if (r >= L) { tk[h] = false; continue; }
          const int u = q.li[i][r];
          tot += (double)q.lv[i][r];
          flat = flat * M + u;
          uu |= u << (8 * i);
        }
      }
      if (tk[h]) {
        tv[h] = tot == tot ? tot : -INFINITY;                        // inf - inf
        tf[h] = flat; tu[h] = uu;
        lv[h] = a.alive == nullptr || a.alive[flat] != 0;
      }
      q.tot[p] = tv[h];
      q.flat[p] = tf[h];
    }
  }
  wave_lds_sync();
  int rc[2] = {0, 0};
#pragma unroll 8
  for (int o = 0; o < cnt; ++o) {
    const double v = q.tot[o];
    rc[0] += v > tv[0];
    rc[1] += v > tv[1];
  }
  auto put_cells = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (tk[h] && rc[h] < K1) {
        q.rf[rc[h]] = tf[h] | (lv[h] ? RANK_LIVE : 0);
        q.ru[rc[h]] = tu[h];
        q.own[rc[h]] = lane + 64 * h;
      }
    wave_lds_sync();
  };
  put_cells();
  clash = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) clash |= tk[h] && rc[h] < K1 && q.own[rc[h]] != lane + 64 * h;
  if (__ballot(clash)) {                                             // equal totals: by flat index
    for (int o = 0; o < cnt; ++o) {
      const double v = q.tot[o];
      const int fo = q.flat[o];
      rc[0] += (v == tv[0]) & (fo < tf[0]);
      rc[1] += (v == tv[1]) & (fo < tf[1]);
    }
    put_cells();
  }
  if constexpr (ALIVE) {
    // the first k alive of the K1 ranked cells, in order
    const int cf = lane < K1 ? q.rf[lane] : 0, cuu = lane < K1 ? q.ru[lane] : 0;
    const uint64_t am = __ballot(lane < K1 && (cf & RANK_LIVE));
    full |= __popcll(am) < k;
    const int pos = __popcll(am & ((1ull << lane) - 1ull));
    if ((am >> lane) & 1ull) { q.rf[pos] = cf; q.ru[pos] = cuu; }
    wave_lds_sync();
  }
  if (full) rank_all_wave<ALIVE>(a, q.dec, M4, q.rf, q.ru);
  const int fl = lane < k ? q.rf[lane] : 0, uu = lane < k ? q.ru[lane] : 0;
  const int f = fl & (RANK_LIVE - 1);
  // Eq. 1 weights from the fp64 totals of the chosen experts, over the alive ones: lane j
  // holds the j-th, sums in slot order
  const bool live = (fl & RANK_LIVE) != 0;
  double gx = 0.0;
#pragma unroll
  for (int i = 0; i < DMAX; ++i) if (i < d) gx += sc[i * M + ((uu >> (8 * i)) & 0xff)];
  double m = live ? gx : -1.0e308;
#pragma unroll
  for (int o = 1; o < KMAX; o <<= 1) {
    const double om = __shfl_xor(m, o, 64);
    m = om > m ? om : m;
  }
  const float ex = live ? expf((float)(gx - m)) : 0.f;
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) sum += __shfl(ex, j, 64);
  const bool any = (__ballot(live) & 0xffull) != 0ull;
  if (lane < k) {
    a.idx[(int64_t)t * k + lane] = f;
    a.w[(int64_t)t * k + lane] = any ? ex / sum : 0.f;
    if (a.g) a.g[(int64_t)t * k + lane] = (float)gx;
  }
}

// Exact fp64 scores S[c] = sum_k x_k W[c][k] + b[c] of one bf16 token by a block of GX_NT
// threads.  Wave w owns the gate columns [w cpw, (w+1) cpw), cpw = ceil(dM / 8), GX_CT at a
// time; lane l sums the 16-byte vectors l, l + 64, ... of the rows (each wave load is 1 KB
// of one row) with fp64 FMAs of the exact element values, GX_P vectors' loads issued before
// any is used; a shuffle tree adds the 64 lane sums.
constexpr int GX_CT = 4;          // gate columns per wave pass
constexpr int GX_P = 3;           // 16-byte vectors in flight
__device__ __forceinline__ void exact_scores(const GateArgs& a, int t, double* s64) {
  using E = bf16;
  constexpr int TB = 1, P = GX_P;
  const int tok[1] = {t};
  constexpr int VEC = 16 / sizeof(E);
  constexpr int NW = GX_NT / 64;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cpw = (a.dM + NW - 1) / NW;
  const int cend = min(a.dM, (w + 1) * cpw);
  const int nv = a.D / VEC;
  const E* x = reinterpret_cast<const E*>(a.x);
  const E* W = reinterpret_cast<const E*>(a.Wg);
  const E* bg = reinterpret_cast<const E*>(a.bg);
  for (int c0 = w * cpw; c0 < cend; c0 += GX_CT) {
    const E* wr[GX_CT];
    const E* xr[TB];
#pragma unroll
    for (int c = 0; c < GX_CT; ++c) wr[c] = W + (int64_t)min(c0 + c, a.dM - 1) * a.D;
#pragma unroll
    for (int t = 0; t < TB; ++t) xr[t] = x + (int64_t)tok[t] * a.D;
    double acc[TB][GX_CT];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int c = 0; c < GX_CT; ++c) acc[t][c] = 0.0;
    for (int v0 = lane; v0 < nv; v0 += 64 * P) {
      uint4 wv[P][GX_CT], xv[P][TB];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int64_t v = v0 + 64 * p;
        if (v < nv) {
#pragma unroll
          for (int c = 0; c < GX_CT; ++c) wv[p][c] = *reinterpret_cast<const uint4*>(wr[c] + v * VEC);
#pragma unroll
          for (int t = 0; t < TB; ++t) xv[p][t] = *reinterpret_cast<const uint4*>(xr[t] + v * VEC);
        }
      }
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (v0 + 64 * p < nv) {
#pragma unroll
          for (int q = 0; q < VEC; ++q) {
            double xd[TB], wd[GX_CT];
#pragma unroll
            for (int t = 0; t < TB; ++t) xd[t] = (double)vec_elem<E>(xv[p][t], q);
#pragma unroll
            for (int c = 0; c < GX_CT; ++c) wd[c] = (double)vec_elem<E>(wv[p][c], q);
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
              for (int c = 0; c < GX_CT; ++c) acc[t][c] = fma(xd[t], wd[c], acc[t][c]);
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TB; ++t) {
#pragma unroll
      for (int c = 0; c < GX_CT; ++c) {
        double v = acc[t][c];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0 && c0 + c < cend) s64[c0 + c] = v + (bg ? (double)ldf(bg + c0 + c) : 0.0);
      }
    }
  }
}

// The tokens the certificate rejects (bf16 MFMA scores): persistent blocks over the queue,
// one token a pass (lowest latency), two blocks per compute unit: 128 registers, of which the
// scores' loads and the selection take all (6 spill with ALIVE, 4 without, outside the score
// loop's loads: the call takes 17-20 us for the wide workload's queue with them).
template <bool ALIVE>
__global__ void __launch_bounds__(GX_NT) __attribute__((amdgpu_waves_per_eu(4)))
gate_exact_sparse_kernel(GateArgs a, const int32_t* queue) {
  __shared__ double s64[DM_MAX];
  __shared__ SelectScratch scratch;
  const int n = queue[0];
  for (int qg = blockIdx.x; qg < n; qg += gridDim.x) {
    const int t = queue[GQ_HEAD + qg];
    exact_scores(a, t, s64);
    __syncthreads();
    if (threadIdx.x < 64) select_wave<ALIVE>(a, rank_tuples<ALIVE>(a), s64, scratch, t);
    else if (threadIdx.x < 128 && a.scores)
      for (int c = threadIdx.x - 64; c < a.dM; c += 64) a.scores[(int64_t)t * a.dM + c] = (float)s64[c];
    __syncthreads();                                                 // s64 reused by the next pass
  }
}

// ---------------------------------------------------------------- exact scores of every token
//
// fp64 scores on v_mfma_f64_16x16x4_f64: the products of fp32 (or bf16) values are exact in
// fp64 and are summed there.  A block scores GF_TOK tokens against all d*M columns: wave wv
// takes the 16 columns of tile wv % CTN over slice wv / CTN of d_model, the slices' sums meet
// in LDS in slice order, and then each wave selects for its tokens.  Lane (r = lane % 16,
// g = lane / 16) loads 16 bytes of row r at vector g of a chunk (4 vectors: 32 bf16 or 16
// fp32 values), for x and Wg alike, and MFMA j of the chunk contracts element j of the four
// vectors; GF_P chunks are loaded one step ahead.  Operands go from memory to registers; the
// tiles' waves share a row of x through the caches, Wg comes from L2 once per 16 tokens.
// Bound by the f64 matrix rate (78.6 TFLOP/s nominal; one MFMA 64 cycles) when T d M D is
// large, else by latency: the first loads, then the selection.  Measured against the scalar
// fp64 kernel it replaces (operands as fp64 in LDS, one lane per token selecting): T = 16384,
// D = 1024, 128 columns, k = 8 355 -> 124 us (55 us of MFMAs); fp32 T = 2048, D = 512, 8
// columns 53 -> 11 us.
constexpr int GF_TOK = 16;        // tokens per block (one MFMA tile)
constexpr int GF_P = 4;           // chunks per step

typedef double f64x4_t __attribute__((ext_vector_type(4)));

//
// LANE: one lane per token selects (select_token; its few undecided tokens go to select_wave),
// in blocks of two token tiles and a wave per tile of columns and tokens.  The least work per
// token, for calls of many tokens with few candidates (gate_route).
template <typename E, bool ALIVE, bool LANE>
__global__ void __launch_bounds__(LANE ? 512 : 1024) gate_topk_f64(GateArgs a, int CTN) {
  extern __shared__ __align__(16) unsigned char sm[];
  constexpr int VEC = 16 / sizeof(E), CHUNK = 4 * VEC;
  const int dM = a.dM, SLD = dM + 1;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int TOK = LANE ? 2 * GF_TOK : GF_TOK;
  const int NWV = blockDim.x >> 6, S = LANE ? 1 : NWV / CTN;
  double* s64 = reinterpret_cast<double*>(sm);                                   // [TOK][SLD]
  // the waves' partial sums, and in their place afterwards the waves' selection scratch
  double (*part)[GF_TOK][17] = reinterpret_cast<double (*)[GF_TOK][17]>(s64 + TOK * SLD);
  SelectScratch& scratch = reinterpret_cast<SelectScratch*>(s64 + TOK * SLD)[wv];
  const int t0 = blockIdx.x * TOK;
  const int r16 = lane & 15, g = lane >> 4;
  const int ct = wv % CTN, sl = LANE ? 0 : wv / CTN;
  const int row = LANE ? wv / CTN * GF_TOK + r16 : r16;
  const RankTuples tup = rank_tuples<ALIVE>(a);
  const E* xr = reinterpret_cast<const E*>(a.x) + (int64_t)min(t0 + row, a.T - 1) * a.D + g * VEC;
  const E* wr = reinterpret_cast<const E*>(a.Wg) + (int64_t)min(16 * ct + r16, dM - 1) * a.D + g * VEC;
  const int nc = a.D / CHUNK;                          // D is a multiple of 64
  const int c0 = nc * sl / S, c1 = nc * (sl + 1) / S;  // this wave's chunks
  f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
  uint4 cx[GF_P], cw[GF_P], nx[GF_P], nw[GF_P];
  auto load = [&](uint4 (&fx)[GF_P], uint4 (&fw)[GF_P], int cc) {
#pragma unroll
    for (int p = 0; p < GF_P; ++p)
      if (cc + p < c1) {
        fx[p] = *reinterpret_cast<const uint4*>(xr + (int64_t)(cc + p) * CHUNK);
        fw[p] = *reinterpret_cast<const uint4*>(wr + (int64_t)(cc + p) * CHUNK);
      }
  };
  load(cx, cw, c0);
  for (int cc = c0; cc < c1; cc += GF_P) {
    load(nx, nw, cc + GF_P);
#pragma unroll
    for (int p = 0; p < GF_P; ++p) {
      if (cc + p < c1) {
#pragma unroll
        for (int j = 0; j < VEC; ++j)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)vec_elem<E>(cw[p], j), (double)vec_elem<E>(cx[p], j), acc,
                                                     0, 0, 0);
      }
    }
#pragma unroll
    for (int p = 0; p < GF_P; ++p) { cx[p] = nx[p]; cw[p] = nw[p]; }
  }
  // element v of the accumulator: column 4 v + lane / 16 of the tile, token lane % 16
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wv][r16][4 * v + g] = acc[v];
  __syncthreads();
  const int nt = min(TOK, a.T - t0);
  {
    const E* bg = reinterpret_cast<const E*>(a.bg);
    const int tok = threadIdx.x & (TOK - 1), half = LANE ? tok / GF_TOK : 0;
    for (int c = threadIdx.x / TOK; c < dM; c += NWV * 64 / TOK) {
      double v = bg ? (double)ldf(bg + c) : 0.0;
      for (int q = 0; q < S; ++q) v += part[(c >> 4) + CTN * (q + half)][tok & (GF_TOK - 1)][c & 15];
      s64[tok * SLD + c] = v;
      if (a.scores && tok < nt) a.scores[(int64_t)(t0 + tok) * dM + c] = (float)v;
    }
  }
  __syncthreads();
  if constexpr (LANE) {
    if (wv > 0) return;
    bool ok = true;
    if (lane < nt)
      ok = select_token<false, true>(s64 + lane * SLD, nullptr, a.alive, a.d, a.M, a.k, a.N, 0.f,
                               a.idx + (int64_t)(t0 + lane) * a.k, a.w + (int64_t)(t0 + lane) * a.k,
                               a.g ? a.g + (int64_t)(t0 + lane) * a.k : nullptr);
    for (uint64_t bad = __ballot(!ok); bad; bad &= bad - 1) {
      const int tt = __builtin_ctzll(bad);
      select_wave<false>(a, tup, s64 + tt * SLD, scratch, t0 + tt);
    }
  } else {
    for (int tt = wv; tt < nt; tt += NWV) select_wave<ALIVE>(a, tup, s64 + tt * SLD, scratch, t0 + tt);
  }
}

// 16-column tiles of the gate columns (at most 8), and waves per block: every tile over as
// many d_model slices as 8 waves allow, or 16 while the blocks are no more than the 256
// compute units (the chain over a slice of d_model and the selections a wave does one after another
// are then the whole call, and both halve).  Measured with 8 / 16 waves: T = 1, D = 4096, 96
// columns 94 / 69 us; T = 200, D = 8192, 96 columns 194 / 140 us; T = 1024, 15625 experts, a
// fifth of them alive, k = 8 340 / 192 us; T = 4096, D = 1024, 64 columns 23 / 21 us.
static int gate_f64_tiles(const Shape& s) { return (int)((s.dM + 15) / 16); }
static int gate_f64_block_waves(const Shape& s) {
  const int n = gate_f64_tiles(s);
  return n * (((s.T + GF_TOK - 1) / GF_TOK <= 256 ? 16 : 8) / n);
}

// The routes of a gate call, all with the same choice of experts: exact scores with a wave per
// token selecting (every shape); for fp32 up to 64 columns also with a lane per token; for bf16
// up to 96 columns also the certified route (three launches: queue clearing, scoring,
// recomputation), unless DMOE_FLAG_GATE_EXACT.
// The route with the lowest estimate is taken.  An estimate is a chain of latencies (the loads
// of d_model, a lane's selection) or the work of all tokens, whichever is longer, with a soft
// corner, plus a start; T and D in thousands, us.  A lane's selection inserts every column into
// lists of `cap` places, then every candidate cell: cap d M and cap x cells steps.  The coefficients
// are least-squares fits to 8100 calls in each route: 12 grids of 2 to 128 columns, d_model 64
// to 4096, 2048 to 65536 tokens, k = 1, 2, 4, 8, bf16 plain and alive-first (nine of ten experts
// alive), fp32 plain; those within a factor of 2.5 of another route count.
// The choice is 0 to 5% above the best route (geometric means).  Lines on T and T d M D in its
// place were 3 to 10% above it and, for narrow d_model, up to 3.3 times as slow as the certified
// route.  Certified / wave / lane, us:
//   bf16, d M = 2: T = 32768, D = 64, k = 1 10 / 33; T = 8192, D = 2048 20 / 21
//   bf16, 2 x 16, k = 4: T = 4096, D = 1024 33 / 14; T = 16384 33 / 41; T = 32768, D = 64 28 / 38
//   bf16, 4 x 8, k = 4: T = 16384, D = 64 35 / 23; D = 2048 53 / 65
//   fp32, 2 x 2, k = 2: T = 8192, D = 64 - / 11 / 7; T = 16384, D = 512 - / 23 / 19, D = 2048 - / 45 / 57
//   fp32, 2 x 32, k = 2: T = 8192, D = 64 - / 13 / 16; T = 65536, D = 512 - / 186 / 157
// Alive-first the certified route depends on how many experts are alive, which the host does
// not know (each token with fewer than k alive among its best cells is computed again: two
// experts of which one is alive, k = 2, 18859 tokens 277 us, 20 with a wave per token), so there
// it has to be the shorter one by a tenth.  A wave per token runs in rounds of two blocks to a
// unit: a last round of a few tokens takes as long as one of half the blocks (D = 64, two columns,
// 8192 tokens 10.7 us, 8330 15.5, 12288 14.8).
enum GateRoute { GR_CERTIFIED, GR_WAVE, GR_LANE };
static double soft_max(double a, double b) {
  a *= a; b *= b;
  return std::sqrt(std::sqrt(a * a + b * b));
}
static GateRoute gate_route(const Shape& s) {
  static constexpr RankTable cells = make_rank_table();
  const bool b16 = s.dtype == DMOE_BF16, alive = (s.flags & DMOE_FLAG_ALIVE_TOPK) != 0;
  const bool cert = b16 && s.dM <= 3 * 32 && !(s.flags & DMOE_FLAG_GATE_EXACT);
  const bool lane = !b16 && !alive && s.dM <= 64 && s.D <= 1024;
  if (!cert && !lane) return GR_WAVE;
  const double T = (double)s.T * 1e-3, D = (double)s.D * 1e-3, dM = (double)s.dM;
  constexpr int64_t round = 2 * 256 * GF_TOK;
  const int64_t last = s.T % round;
  const double Tw = s.T > round && last > 0 && last < round / 2 ? (double)(s.T - last + round / 2) * 1e-3 : T;
  const int n = gate_f64_tiles(s), te = n <= 2 ? n : n <= 4 ? 4 : 8;        // waves a tile of columns occupies
  const double chain = D * te / ((s.T + GF_TOK - 1) / GF_TOK <= 256 ? 16 : 8);
  const int cap = alive ? (s.k <= 4 ? 7 : KMAX + 3) : (s.k <= 4 ? 5 : KMAX + 1);
  const int K1 = (int)std::min<int64_t>(s.N, alive ? cap : s.k + 1);
  const double cols = 0.01 * cap * dM, cell = 0.01 * cap * (double)std::min<int64_t>(s.N, cells.cnt[s.d - 1][K1]);
  if (lane) {
    const double w = soft_max(3.99 + 55.7 * chain, Tw * (0.775 + 0.818 * D * te + 0.00592 * dM)) + 3.98;
    const double l = soft_max(17.7 * D + 3.07 * cols + 11.8 * cell, T * (0.0422 + 0.953 * D * te + 0.155 * (cols + cell))) + 3.6;
    return l < w ? GR_LANE : GR_WAVE;
  }
  const int CB = (int)((s.dM + 31) / 32);
  const double De = D / gm_kw(s.D);
  double w, c;
  if (!alive) {
    w = 1.05 * (soft_max(4.18 + 42.0 * chain, Tw * (0.798 + 0.624 * D * te + 0.00593 * dM)) + 3.94);
    c = soft_max(3.6 + De * (2.83 + 7.59 * CB) + 3.79 * cols + 13.6 * cell,
                 T * (D * (0.13 + 0.372 * CB) + 0.131 * (cols + cell))) + 7.02;
  } else {
    w = 0.9 * (soft_max(3.96 + 44.1 * chain, Tw * (0.902 + 0.628 * D * te + 0.0104 * dM)) + 4.63);
    c = soft_max(8.03 + De * (2.38 + 8.07 * CB) + 3.29 * cols + 17.4 * cell,
                 T * (D * (0.277 + 0.324 * CB) + 0.206 * (cols + cell)));
  }
  return c < w ? GR_CERTIFIED : GR_WAVE;
}
static int gate_f64_tokens(bool lane) { return lane ? 2 * GF_TOK : GF_TOK; }
static int gate_f64_waves(const Shape& s, bool lane) { return lane ? gate_f64_tiles(s) * 2 : gate_f64_block_waves(s); }
static size_t gate_f64_lds_bytes(const Shape& s, bool lane) {
  static_assert(GF_TOK % 2 == 0 && alignof(SelectScratch) <= 16, "s64 rows end on 16 bytes");
  const size_t part = GF_TOK * 17 * sizeof(double);
  return gate_f64_tokens(lane) * (s.dM + 1) * sizeof(double) + gate_f64_waves(s, lane) * std::max(part, sizeof(SelectScratch));
}
static size_t gate_mfma_lds_bytes(int dM, int kw) {
  const size_t ring = (size_t)kw * GM_RING * 4096 * (1 + (dM + 31) / 32);
  const size_t scores = (sizeof(double) + sizeof(float)) * GM_TOK * (dM + 1);
  return ring > scores ? ring : scores;
}

// ---------------------------------------------------------------- backward
//
// dg[t,j] = w (dw - sum_l w_l dw_l) over alive chosen experts; ds row t gets dg at column
// i*M + u_i for every dimension i; dWg = ds^T x, dbg = sum_t ds.  Two launches: one kernel
// whose blocks either write dg and the bias gradient's partial sums (GD_TOK tokens each) or
// multiply a token split by GB_BN columns of x into a partial dWg, and a reduction of the
// partials in split order.  Every block of the first launch reads w and dw, so when dg lies
// over one of them the second launch writes it instead (the call is then 2.8 us longer at
// k = 8: the tokens' loads and arithmetic once more).
// ds is never stored: a block expands the k terms per token and dimension of the tokens of its
// next stage in LDS, column-major like an MFMA operand.  A thread owns one token's entries of
// one dimension: it clears those it wrote two stages ago and writes the new ones, so the
// expansion needs no barrier of its own.  bf16: ds as hi and lo bf16 parts, both multiplied
// into the same fp32 accumulator (about 16 mantissa bits).
// Bound by latency: a stage's expansion, barrier and loads follow one another, two blocks to
// a compute unit (T = 32768, D = 4096, 32 columns: 92 us for 268 MB, 2.9 TB/s).  Five
// launches before (dg and dense ds; split offsets; a register-staged GEMM over ds in memory;
// two reductions), measured before -> now per call: that shape 170 -> 97 us; T = 16384,
// D = 1024, 128 columns, k = 8 130 -> 48 us; T = 4096, D = 1024, 64 columns 67 -> 18 us;
// fp32 T = 2048, D = 512, 8 columns 79 -> 19 us.

constexpr int GB_NT = 256;
constexpr int GB_BN = 128;         // x columns per block, 32 per wave
constexpr int GB_ST = 3;           // x stages in LDS
constexpr int GB_XB = 16384;       // bytes of an x stage: 64 bf16 or 32 fp32 rows

struct GateBwdArgs {
  const void* x; const int32_t* idx; const float* w; const float* dw; const uint8_t* alive;
  float* dg; float* dbg_part; float* part;
  int T, D, d, M, k, dM;
  int gblk, nb, split;             // dg blocks; column blocks; tokens per split
  int dg_late;                     // dg is written by the second launch
};

// The k terms of token t: dg and the grid indices (8 bits per dimension); zeros past `end`.
struct GateTerms {
  int id[KMAX];
  float wv[KMAX], dv[KMAX];
  uint8_t live[KMAX];
  // the slots' loads; the alive flags, which need the ids, are loaded by a second call
  __device__ __forceinline__ void load(const GateBwdArgs& p, int t, int end) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      id[j] = 0; wv[j] = 0.f; dv[j] = 0.f;
      if (j < p.k && t < end) {
        id[j] = p.idx[(int64_t)t * p.k + j];
        wv[j] = p.w[(int64_t)t * p.k + j];
        dv[j] = p.dw[(int64_t)t * p.k + j];
      }
    }
  }
  __device__ __forceinline__ void load_alive(const GateBwdArgs& p) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      live[j] = 1;
      if (j < p.k && p.alive != nullptr) live[j] = p.alive[id[j]];
    }
  }
  // f(j, dg, indices) for each slot
  template <typename F> __device__ __forceinline__ void each(const GateBwdArgs& p, F&& f) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (j < p.k) {
        if (live[j] == 0) wv[j] = 0.f;
        s = fmaf(wv[j], dv[j], s);
      }
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (j < p.k) {
        int rem = id[j];
        uint32_t dig = 0;
#pragma unroll
        for (int i = DMAX - 1; i >= 0; --i)
          if (i < p.d) { dig |= (uint32_t)(rem % p.M) << (8 * i); rem /= p.M; }
        f(j, wv[j] * (dv[j] - s), dig);
      }
  }
};

// dg of GD_TOK tokens (unless it is left to the second launch), and their sums per gate column
// (rows in order, in two halves)
__device__ __forceinline__ void gate_dg_block(const GateBwdArgs& p, int blk, float* rows) {
  const int SR = p.dM + 1;
  const int t0 = blk * GD_TOK, nt = min(GD_TOK, p.T - t0);
  for (int q = threadIdx.x; q < GD_TOK * SR; q += GB_NT) rows[q] = 0.f;
  __syncthreads();
  if ((int)threadIdx.x < nt) {
    const int t = t0 + threadIdx.x;
    GateTerms v;
    v.load(p, t, p.T);
    v.load_alive(p);
    float* row = rows + threadIdx.x * SR;
    v.each(p, [&](int j, float g, uint32_t dig) {
      if (!p.dg_late) p.dg[(int64_t)t * p.k + j] = g;
      for (int i = 0; i < p.d; ++i) row[i * p.M + ((dig >> (8 * i)) & 0xff)] += g;
    });
  }
  if (!p.dbg_part) return;
  __syncthreads();
  const int c = threadIdx.x >> 1;                        // dM <= 128 = GB_NT / 2
  float s = 0.f;
  if (c < p.dM) {
    const float* col = rows + (threadIdx.x & 1) * (GD_TOK / 2) * SR + c;
#pragma unroll 8
    for (int r = 0; r < GD_TOK / 2; ++r) s += col[r * SR];
  }
  s += __shfl_xor(s, 1, 64);
  if (c < p.dM && (threadIdx.x & 1) == 0) p.dbg_part[(int64_t)blk * p.dM + c] = s;
}

template <typename E> struct GbTile;     // the x stage: [tokens][GB_BN columns]
template <> struct GbTile<bf16> { using X = NcTile<GB_BN, GB_NT / 64, 64>; static constexpr int TOK = 64, PARTS = 2; };
template <> struct GbTile<float> { using X = NcTileF32<GB_BN, GB_NT / 64>; static constexpr int TOK = 32, PARTS = 1; };

template <typename E, int CB>      // CB: 32-column blocks of the d*M gate columns
__global__ void __launch_bounds__(GB_NT) gate_bwd_kernel(GateBwdArgs p) {
  using X = typename GbTile<E>::X;
  using KC = KcTile<32, 4, 1, 64>;                       // fragment layout of a 128-byte ds row
  constexpr int TOK = GbTile<E>::TOK, PARTS = GbTile<E>::PARTS;
  constexpr int SPC = GB_NT / TOK;                       // stages per GB_NT tokens
  constexpr int DSB = 32 * CB * 128;                     // bytes of one ds part: [32 CB][TOK]
  static_assert(X::BYTES == GB_XB && X::INSTR % (GB_NT / 64) == 0, "x stage");
  extern __shared__ __align__(1024) char smem[];
  if ((int)blockIdx.x < p.gblk) {
    gate_dg_block(p, blockIdx.x, reinterpret_cast<float*>(smem));
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x - p.gblk;
  const int n0 = (b % p.nb) * GB_BN, sp = b / p.nb;
  const int tb = sp * p.split, te = min(p.T, tb + p.split);
  const int nk = (te - tb + TOK - 1) / TOK;
  const E* x = reinterpret_cast<const E*>(p.x) + (int64_t)tb * p.D + n0;
  char* dsb = smem + GB_ST * GB_XB;                      // 2 x PARTS x DSB
  uint2* terms = reinterpret_cast<uint2*>(dsb + 2 * PARTS * DSB);   // [k][GB_NT]: dg, indices
  for (int q = tid; q < 2 * PARTS * DSB / 16; q += GB_NT) reinterpret_cast<uint4*>(dsb)[q] = make_uint4(0, 0, 0, 0);

  auto issue = [&](int kt) {
    X::load(x + (int64_t)kt * TOK * p.D, p.D, p.D - n0, te - tb - kt * TOK, smem + (kt % GB_ST) * GB_XB, wave, lane);
  };
  GateTerms v;
  auto put_terms = [&]() {
    v.each(p, [&](int j, float g, uint32_t dig) { terms[j * GB_NT + tid] = make_uint2(__float_as_uint(g), dig); });
  };
  // this thread's token and dimension of a stage, and the column of each slot it wrote last
  // into either ds buffer
  const int bt = tid % TOK, bi = tid / TOK;
  const bool builder = bi < p.d;
  uint8_t old[2][KMAX];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int j = 0; j < KMAX; ++j) old[q][j] = 0;
  auto ds_at = [&](char* base, int c) -> E* {            // element (column c, token bt)
    constexpr int PER = 16 / (int)sizeof(E);
    return reinterpret_cast<E*>(base + c * 128 + (((bt / PER) ^ ((c >> 1) & 7)) << 4)) + bt % PER;
  };
  auto build = [&](int kt, auto BUFc) {
    constexpr int BUF = decltype(BUFc)::value;
    if (!builder) return;
    char* hi = dsb + BUF * PARTS * DSB;
    const uint2* tt = terms + (kt % SPC) * TOK + bt;
    float g[KMAX];
    int c[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      g[j] = 0.f;
      c[j] = -1;
      if (j < p.k) {
        const uint2 q = tt[j * GB_NT];
        g[j] = __uint_as_float(q.x);
        c[j] = bi * p.M + (int)((q.y >> (8 * bi)) & 0xff);
        *ds_at(hi, old[BUF][j]) = 0;
        if constexpr (PARTS == 2) *ds_at(hi + DSB, old[BUF][j]) = 0;
      }
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (j >= p.k) continue;
      float s = 0.f;                                     // every slot of the column, in slot order
#pragma unroll
      for (int l = 0; l < KMAX; ++l) s += c[l] == c[j] ? g[l] : 0.f;
      if constexpr (PARTS == 2) {
        const bf16 h = f2bf(s);
        *ds_at(hi, c[j]) = h;
        *ds_at(hi + DSB, c[j]) = f2bf(s - bf2f(h));
      } else {
        *ds_at(hi, c[j]) = s;
      }
      old[BUF][j] = (uint8_t)c[j];
    }
  };
  uint32_t kc_off[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) kc_off[q] = KC::lane_off(2 * q, lane);
  const uint32_t x_off = X::lane_off(wave, lane);
  f32x16_t acc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;

  v.load(p, tb + tid, te);
  v.load_alive(p);
  put_terms();
#pragma unroll
  for (int st = 0; st < GB_ST - 1; ++st)
    if (st < nk) issue(st);
  block_sync_lds();
  // the old columns start as column 0 of dimension 0, which only its own builder may write:
  // clears before the first build of a buffer must not race with it
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int j = 0; j < KMAX; ++j) old[q][j] = (uint8_t)(builder ? bi * p.M : 0);
  build(0, std::integral_constant<int, 0>{});
  if (SPC < nk) v.load(p, tb + GB_NT + tid, te);

  auto stage = [&](int kt, auto BUFc) {
    constexpr int BUF = decltype(BUFc)::value;           // kt % 2
    if (kt + GB_ST - 2 < nk) wait_vmcnt<(GB_ST - 2) * X::PER_WAVE>();
    else wait_vmcnt<0>();
    block_sync_lds();              // x and ds of stage kt are whole; every wave is done with stage kt - 1
    // The terms of the next GB_NT tokens: slots loaded SPC stages ahead, their alive flags two
    // stages later, put in LDS when the tokens' first stage is to be built.  These come before
    // the stage's own loads: a wait for a register load also waits for every load before it.
    if (kt % SPC == 1 && kt - 1 + SPC < nk) v.load_alive(p);
    if ((kt + 1) % SPC == 0 && kt + 1 < nk) {
      put_terms();                 // every build of the previous tokens is done
      block_sync_lds();
      if (kt + 1 + SPC < nk) v.load(p, tb + (kt + 1 + SPC) * TOK + tid, te);
    }
    if (kt + GB_ST - 1 < nk) issue(kt + GB_ST - 1);
    if (kt + 1 < nk) build(kt + 1, std::integral_constant<int, 1 - BUF>{});
    const char* xs = smem + (kt % GB_ST) * GB_XB;
    const char* ds = dsb + BUF * PARTS * DSB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (sizeof(E) == 2) {
        const bf16x8_t fx = X::frag_at(xs, q * 16, x_off);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, KC::frag_at(ds, cb * 32, kc_off[q]), acc[cb], 0, 0, 0);
          acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, KC::frag_at(ds + DSB, cb * 32, kc_off[q]), acc[cb], 0, 0, 0);
        }
      } else {
        const f32x4_t fx = frag_f32<true, X>(xs, q, 0, x_off);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const f32x4_t fd = frag_f32<false, KC>(ds, q, cb * 32, kc_off[q]);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(fx[r], fd[r], acc[cb], 0, 0, 0);
        }
      }
    }
  };
  for (int kt = 0; kt < nk; kt += 2) {
    stage(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < nk) stage(kt + 1, std::integral_constant<int, 1>{});
  }
  // lane (column l % 32 of each block, half l / 32) holds x columns 8 g + 4 (l / 32) .. + 3
  const int l32 = lane & 31, lhi = lane >> 5;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int c = cb * 32 + l32;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = n0 + wave * 32 + 8 * g + 4 * lhi;
      if (c < p.dM && n < p.D)
        *reinterpret_cast<float4*>(p.part + ((int64_t)sp * p.dM + c) * p.D + n) =
            make_float4(acc[cb][4 * g], acc[cb][4 * g + 1], acc[cb][4 * g + 2], acc[cb][4 * g + 3]);
    }
  }
}

static size_t gate_bwd_lds_bytes(const Shape& s) {
  const int parts = s.dtype == DMOE_BF16 ? 2 : 1;
  const size_t ds = (size_t)2 * parts * ((s.dM + 31) / 32) * 32 * 128;
  const size_t mm = (size_t)GB_ST * GB_XB + ds + (size_t)s.k * GB_NT * sizeof(uint2);
  const size_t rows = (size_t)GD_TOK * (s.dM + 1) * sizeof(float);
  return mm > rows ? mm : rows;
}

// dWg = sum of the splits' partials in split order (4 values a thread); the ndg blocks past
// nred: dg, a token a thread; the blocks past those: dbg[c] = sum over the dg blocks of their
// partial column sums, thread i adding a contiguous run of blocks, then a tree over the
// threads.
template <typename E>
__global__ void __launch_bounds__(256)
gate_reduce_kernel(GateBwdArgs p, int nsplit, int64_t n, E* dWg, int nred, int ndg, E* dbg) {
  const float* part = p.part;
  const float* dbg_part = p.dbg_part;
  const int nblk = p.gblk, dM = p.dM;
  if ((int)blockIdx.x < nred) {
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (q >= n) return;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int sp = 0; sp < nsplit; ++sp) {
      const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)sp * n + q);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    // dWg needs no alignment beyond its elements'
    dWg[q] = cvt<E>(s.x); dWg[q + 1] = cvt<E>(s.y); dWg[q + 2] = cvt<E>(s.z); dWg[q + 3] = cvt<E>(s.w);
    return;
  }
  if ((int)blockIdx.x < nred + ndg) {
    const int t = ((int)blockIdx.x - nred) * 256 + (int)threadIdx.x;
    GateTerms v;
    v.load(p, t, p.T);
    v.load_alive(p);
    if (t < p.T) v.each(p, [&](int j, float g, uint32_t) { p.dg[(int64_t)t * p.k + j] = g; });
    return;
  }
  const int c = blockIdx.x - nred - ndg;
  const int per = (nblk + 255) / 256;
  const int b0 = threadIdx.x * per, b1 = min(nblk, b0 + per);
  float s = 0.f;
  for (int b = b0; b < b1; ++b) s += dbg_part[(int64_t)b * dM + c];
  __shared__ float red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) dbg[c] = cvt<E>(red[0]);
}

}  // namespace dmoe

using namespace dmoe;

extern "C" int dmoe_gate_topk(const dmoe_dims* dims, const void* x, const void* Wg, const void* bg,
                              const uint8_t* alive, int32_t* idx, float* w, float* g, float* scores,
                              void* ws, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (s.T == 0) return DMOE_OK;
  if (!x || !Wg || !idx || !w) return DMOE_EINVAL;
  if (!aligned16(x) || !aligned16(Wg)) return DMOE_EUNSUPPORTED;
  GateArgs a{x, Wg, bg, alive, idx, w, g, scores, (int)s.T, (int)s.D, s.d, s.M, s.k, (int)s.dM, (int)s.N};
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const bool alive_first = (s.flags & DMOE_FLAG_ALIVE_TOPK) != 0;
  const bool mfma = s.dtype == DMOE_BF16 && s.dM <= 3 * 32;
  if (mfma || alive_first) {
    if (!ws) return DMOE_EINVAL;
    if (!aligned16(ws)) return DMOE_EUNSUPPORTED;
  }
  const GateRoute route = gate_route(s);
  if (route != GR_CERTIFIED) {
    // exact fp64 scores for every token
    const bool lane = route == GR_LANE;
    const int tok = gate_f64_tokens(lane);
    const dim3 grid((unsigned)((s.T + tok - 1) / tok));
    auto go = [&](auto EK) {
      using E = typename decltype(EK)::type;
      auto kern = alive_first ? gate_topk_f64<E, true, false> : gate_topk_f64<E, false, false>;
      if constexpr (sizeof(E) == 4)
        if (lane) kern = gate_topk_f64<E, false, true>;
      DMOE_LAUNCH_NAMED("gate_topk_f64", kern, grid, dim3(64 * gate_f64_waves(s, lane)), gate_f64_lds_bytes(s, lane), st, a,
                        gate_f64_tiles(s));
    };
    if (s.dtype == DMOE_BF16) go(type_tag<bf16>{});
    else go(type_tag<float>{});
    return launch_status();
  }
  // error factor of the MFMA scores (see the certificate above gate_topk_mfma)
  const double u = 1.0 / 8388608.0;
  const double g32 = 32 * u / (1 - 32 * u) + (s.D / 32 + 8) * 2.220446049250313e-16;
  const double gD = (double)s.D * u / (1 - (double)s.D * u);
  int32_t* queue = reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(ws) + workspace_layout(s).gq_off);
  GateMfmaArgs ga{a, (float)(g32 / (1 - gD) * 1.0001), queue};
  const int KW = gm_kw(s.D);
  const size_t lds = gate_mfma_lds_bytes((int)s.dM, KW);
  const int CB = (int)((s.dM + 31) / 32);
  auto pick = [&](auto AL) {
    constexpr bool A = decltype(AL)::value;
    return KW == 2 ? (CB == 1 ? gate_topk_mfma<1, 2, A> : CB == 2 ? gate_topk_mfma<2, 2, A> : gate_topk_mfma<3, 2, A>)
                   : (CB == 1 ? gate_topk_mfma<1, 1, A> : CB == 2 ? gate_topk_mfma<2, 1, A> : gate_topk_mfma<3, 1, A>);
  };
  auto kern = alive_first ? pick(std::true_type{}) : pick(std::false_type{});
  if (lds > 65536) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
  }
  fill_zero(queue, sizeof(int32_t), st);
  const dim3 grid((unsigned)((s.T + GM_TOK - 1) / GM_TOK));
  DMOE_LAUNCH_NAMED("gate_topk_mfma", kern, grid, dim3(64 * KW), lds, st, ga);
  // exact recomputation of the queued tokens: persistent blocks over the queue
  const int xgrid = (int)std::min<int64_t>(s.T, 1024);
  if (alive_first) DMOE_LAUNCH(gate_exact_sparse_kernel<true>, dim3(xgrid), dim3(GX_NT), 0, st, a, queue);
  else DMOE_LAUNCH(gate_exact_sparse_kernel<false>, dim3(xgrid), dim3(GX_NT), 0, st, a, queue);
  return launch_status();
}

template <typename E>
static int gate_bwd_impl(const Shape& s, const void* x, const int32_t* idx, const float* w,
                         const float* dw, const uint8_t* alive, float* dg, void* dWg, void* dbg,
                         void* ws, hipStream_t st) {
  const Workspace L = workspace_layout(s);
  unsigned char* base = reinterpret_cast<unsigned char*>(ws);
  GateBwdArgs p{x, idx, w, dw, alive, dg, nullptr, reinterpret_cast<float*>(base + L.part_off),
                (int)s.T, (int)s.D, s.d, s.M, s.k, (int)s.dM,
                (int)((s.T + GD_TOK - 1) / GD_TOK), (int)((s.D + GB_BN - 1) / GB_BN), (int)L.gsplit_tokens, 0};
  auto over = [&](const float* q) {
    const uintptr_t a = (uintptr_t)dg, b = (uintptr_t)q, n = (uintptr_t)s.P * sizeof(float);
    return a < b + n && b < a + n;
  };
  p.dg_late = over(w) || over(dw);
  // the bias gradient's per-block column sums use the forward pass's queue region, which is
  // sized for both (calls on one stream do not overlap)
  if (dbg) p.dbg_part = reinterpret_cast<float*>(base + L.gq_off);
  const size_t lds = gate_bwd_lds_bytes(s);
  auto go = [&](auto CBc) {
    auto kern = gate_bwd_kernel<E, decltype(CBc)::value>;
    if (lds > 65536) {
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      (void)hipGetLastError();
    }
    DMOE_LAUNCH_NAMED("gate_bwd_kernel (dg, dWg per token split)", kern,
                      dim3((unsigned)(p.gblk + p.nb * (int)L.gsplit)), dim3(GB_NT), lds, st, p);
  };
  switch ((s.dM + 31) / 32) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    default: go(std::integral_constant<int, 4>{}); break;
  }
  const int64_t n = s.dM * s.D;                          // a multiple of 64
  const int nred = (int)((n / 4 + 255) / 256), ndg = p.dg_late ? (int)((s.T + 255) / 256) : 0;
  DMOE_LAUNCH_NAMED("gate_reduce_kernel", gate_reduce_kernel<E>, dim3((unsigned)(nred + ndg + (dbg ? s.dM : 0))),
                    dim3(256), 0, st, p, (int)L.gsplit, n, reinterpret_cast<E*>(dWg), nred, ndg,
                    reinterpret_cast<E*>(dbg));
  return launch_status();
}

extern "C" int dmoe_gate_topk_bwd(const dmoe_dims* dims, const void* x, const int32_t* idx,
                                  const float* w, const float* dw, const uint8_t* alive, float* dg,
                                  void* dWg, void* dbg, void* ws, void* stream) {
  Shape s;
  int rc = check_dims(dims, &s);
  if (rc) return rc;
  if (!dWg) return DMOE_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (s.T == 0) {
    // no tokens: zero gradients (a fill kernel, so the call can be graph-captured)
    fill_zero(dWg, (size_t)s.dM * s.D * s.esz, st);
    if (dbg) fill_zero(dbg, (size_t)s.dM * s.esz, st);
    return launch_status();
  }
  if (!x || !idx || !w || !dw || !dg || !ws) return DMOE_EINVAL;
  if (!aligned16(x) || !aligned16(ws)) return DMOE_EUNSUPPORTED;
  if (s.dtype == DMOE_BF16) return gate_bwd_impl<bf16>(s, x, idx, w, dw, alive, dg, dWg, dbg, ws, st);
  return gate_bwd_impl<float>(s, x, idx, w, dw, alive, dg, dWg, dbg, ws, st);
}
