// Grouped fp32 GEMM on v_mfma_f32_32x32x2_f32, fed by the direct global->LDS loads of
// gemm2.hpp (16 bytes per lane, no staging registers) through a ring of STAGES buffers.
//
// Problem statement of gemm.hpp, accumulator layout of gemm2.hpp:
//   C[m][n] = sum_k A[m][k] B[n][k] per expert; GROUP_M groups rows (tokens), GROUP_K
//   groups the contraction (tokens) for weight gradients.
//   A_T / B_T: the operand is stored with m (n) contiguous, one row per k.
//
// What bounds it: one 32x32x2 MFMA takes 64 cycles and reads 8 bytes per lane, so LDS
// bandwidth is far away; the loads have to be in flight early enough, and enough waves
// have to share a SIMD.  A stage is 32 k deep, so a K-contiguous row is 128 bytes and the
// tile has the bytes, and the swizzle, of the bf16 GEMM's 64-deep one; a lane's 16-byte
// read gives it 4 consecutive k, one for each of 4 MFMAs: MFMA j of the 8-k group q
// contracts k = 8q + j (lanes 0-31) and k = 8q + 4 + j (lanes 32-63).  An N-contiguous
// tile is read 4 bytes per lane with the same k order, 32 consecutive lanes on 32
// consecutive banks; rows with k % 8 >= 4 store their 32-column halves exchanged, so that
// the two halves of a wave use different banks.
//
// Measured against the register-staged kernel it replaces (32 x 64 tiles of two waves,
// scalar LDS reads), 8.6 GFLOP a launch: row-grouped 206 to 244 us -> 101 to 110 us,
// weight gradients 202 to 205 us -> 88 to 93 us.  The MFMA pipes are busy 53 to 58% of a
// row-grouped launch and 64% of a weight gradient (counters, 2.4 GHz); the rest is the launch,
// the first stages' latency and the last tiles, which run one to a unit.
#pragma once

#include "gemm2.hpp"

namespace dmoe {

constexpr int F32_BK = 32;       // k per stage

// N-contiguous fp32 tile [32][R]: row k holds R/4 chunks of 16 bytes, chunk c stored at
// position c ^ (8 * ((k / 4) % 2)).
template <int R, int NW>
struct NcTileF32 {
  static constexpr int RB = R * 4;                     // bytes per row
  static constexpr int BYTES = F32_BK * RB;
  static constexpr int CPR = R / 4;                    // chunks per row
  static constexpr int RPI = 1024 / RB;                // rows per wave instruction
  static constexpr int INSTR = F32_BK / RPI;
  static constexpr int PER_WAVE = INSTR / NW;
  static_assert(R == 64 || R == 128, "two or four 32-column blocks");
  static_assert(INSTR % NW == 0, "equal load counts per wave");
  // element (col c, k) at base[k * ld + c]; rows k >= kvalid clamped (zeroed later)
  __device__ __forceinline__ static void load(const float* base, int64_t ld, int cvalid, int kvalid, char* lds,
                                              int wave, int lane) {
    char* lw = lds + wave * 1024;
    static_for<PER_WAVE>([&](auto I) {
      constexpr int i = decltype(I)::value;
      const int k = (wave + i * NW) * RPI + lane / CPR;
      int col = ((lane % CPR) ^ (8 * ((k >> 2) & 1))) * 4;
      col = col < cvalid ? col : ((cvalid - 1) & ~3);
      const int kk = k < kvalid ? k : kvalid - 1;
      g2l_16_at<i * NW * 1024>(reinterpret_cast<const bf16*>(base), ((uint32_t)kk * (uint32_t)ld + (uint32_t)col) * 4u,
                               lw);
    });
  }
  // zero rows [kvalid, kend) of the tile (GROUP_K tail)
  __device__ __forceinline__ static void zero_tail(char* lds, int kvalid, int kend, int tid, int nt) {
    uint4* p = reinterpret_cast<uint4*>(lds + kvalid * RB);
    const int n = (kend - kvalid) * CPR;
    for (int i = tid; i < n; i += nt) p[i] = make_uint4(0, 0, 0, 0);
  }
  // this lane's byte offset in the 32-column block m, for k = 0; the 8-k group q and the
  // MFMA j add (8 q + j) rows
  __device__ __forceinline__ static uint32_t lane_off(int m, int lane) {
    const int h = lane >> 5, l = lane & 31;
    return (uint32_t)(4 * h * RB + ((((8 * m) ^ (8 * h)) + (l >> 2)) << 4) + (l & 3) * 4);
  }
};

// Per-wave fragment of one 32-row block for an 8-k group: 4 values per lane.
template <bool T, typename TILE>
__device__ __forceinline__ f32x4_t frag_f32(const char* tile, int q, int r0, uint32_t off) {
  if constexpr (T) {
    f32x4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const float*>(tile + (8 * q + j) * TILE::RB + off);
    return v;
  } else {
    return *reinterpret_cast<const f32x4_t*>(tile + r0 * TILE::RB + off);
  }
}

template <int GM, bool A_T, bool B_T, int EPI, int BM, int BN, int WM, int WN, int STAGES>
__global__ void __launch_bounds__(64 * WM * WN)
grouped_gemm_f32(GemmArgs<float> p) {
  constexpr int NW = WM * WN, NT = 64 * NW, BK = F32_BK;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  // the K-contiguous tile: rows of 32 floats = 128 bytes, as 64 bf16
  using TA = typename std::conditional<A_T, NcTileF32<BM, NW>, KcTile<BM, NW, 1, 64>>::type;
  using TB = typename std::conditional<B_T, NcTileF32<BN, NW>, KcTile<BN, NW, 1, 64>>::type;
  using KC = KcTile<32, NW, 1, 64>;
  constexpr int SBYTES = TA::BYTES + TB::BYTES;
  constexpr int LPS = TA::PER_WAVE + TB::PER_WAVE;
  static_assert(TM >= 1 && TN >= 1 && STAGES >= 2, "tile");
  static_assert(TA::INSTR % NW == 0 && TB::INSTR % NW == 0, "equal load counts per wave");
  static_assert(GM == GROUP_M ? !A_T : (A_T && B_T), "GROUP_K takes both operands stored per token");

  extern __shared__ __align__(1024) char smem[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, lhi = lane >> 5;

  // per-lane byte offsets of the fragments within a stage
  uint32_t kc_off[BK / 8], a_nc[TM], b_nc[TN];
#pragma unroll
  for (int q = 0; q < BK / 8; ++q) kc_off[q] = KC::lane_off(2 * q, lane);
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    a_nc[j] = 0;
    if constexpr (A_T) a_nc[j] = TA::lane_off(wm * TM + j, lane);
  }
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    b_nc[i] = 0;
    if constexpr (B_T) b_nc[i] = TB::lane_off(wn * TN + i, lane);
  }

  const int total = ld_plan(p.tprefix, p.groups) * p.tscale;
  int L, Lend, Lstep;
  if (p.chunked) {         // each XCD a contiguous share of the tile list (one L2 per slab)
    const int x = blockIdx.x & 7, lb = blockIdx.x >> 3;
    L = (int)(((int64_t)x * total) >> 3) + lb;
    Lend = (int)(((int64_t)(x + 1) * total) >> 3);
    Lstep = (gridDim.x - x + 7) >> 3;
  } else {
    L = blockIdx.x; Lend = total; Lstep = gridDim.x;
  }
  const int NTILES = (p.N + BN - 1) / BN;

  int ehint = 0;
  for (; L < Lend; L += Lstep) {
    const int e = find_group_plan(p.tprefix, p.tscale, p.groups, L, ehint);
    ehint = e;
    const int q0 = L - ld_plan(p.tprefix, e) * p.tscale;
    const int off = ld_plan(p.offsets, e);
    const int cnt = ld_plan(p.offsets, e + 1) - off;
    int m0, n0, mvalid, kvalid;
    const float *Ab, *Bb;
    if constexpr (GM == GROUP_M) {
      const int mt_e = (cnt + BM - 1) / BM;
      m0 = (q0 % mt_e) * BM;
      n0 = (q0 / mt_e) * BN;
      mvalid = cnt - m0;
      kvalid = p.K;
      Ab = p.A + (int64_t)(off + m0) * p.lda;
      Bb = p.B + (int64_t)e * p.b_gstride + (B_T ? (int64_t)n0 : (int64_t)n0 * p.ldb);
    } else {
      m0 = (q0 / NTILES) * BM;
      n0 = (q0 % NTILES) * BN;
      mvalid = p.M - m0;
      kvalid = cnt;
      Ab = p.A + (int64_t)off * p.lda + m0;
      Bb = p.B + (int64_t)off * p.ldb + n0;
    }
    const int nvalid = p.N - n0;
    const int nk = (kvalid + BK - 1) / BK;

    auto issue = [&](int kt) {
      char* buf = smem + (kt % STAGES) * SBYTES;
      const int k0 = kt * BK;
      if constexpr (A_T) TA::load(Ab + (int64_t)k0 * p.lda, p.lda, mvalid, kvalid - k0, buf, wave, lane);
      else TA::load(reinterpret_cast<const bf16*>(Ab + k0), 2 * p.lda, mvalid, buf, wave, lane);
      if constexpr (B_T) TB::load(Bb + (int64_t)k0 * p.ldb, p.ldb, nvalid, kvalid - k0, buf + TA::BYTES, wave, lane);
      else TB::load(reinterpret_cast<const bf16*>(Bb + k0), 2 * p.ldb, nvalid, buf + TA::BYTES, wave, lane);
    };

    f32x16_t acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    block_sync_lds();                    // every wave is done with the previous tile's ring
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nk) issue(s);
    // One stage: wait for it, refill the slot of the stage before it, multiply.  LAST: the
    // tile's last stage (with GROUP_K it may hold less than 32 rows of the expert); LIVE:
    // the wave has a live 32-row block (else it only loads).  Both are compile-time, so the
    // accumulators stay in place through the loop.
    auto stage = [&](int kt, auto LASTc, auto LIVEc) {
      constexpr bool LAST = decltype(LASTc)::value, LIVE = decltype(LIVEc)::value;
      // loads retire in issue order; behind stage kt at most STAGES - 2 stages are issued
      if (!LAST && kt + STAGES - 2 < nk) wait_vmcnt<(STAGES - 2) * LPS>();
      else wait_vmcnt<0>();
      char* buf = smem + (kt % STAGES) * SBYTES;
      const int kv = kvalid - kt * BK;   // rows of the expert in this stage (GROUP_K)
      if constexpr (GM == GROUP_K) {
        // token rows past the expert's last: zeros, up to the end of the 8-k group
        if (LAST && kv < BK) {
          block_sync_lds();              // every wave's loads of this stage have landed
          const int kend = (kv + 7) / 8 * 8;
          TA::zero_tail(buf, kv, kend, tid, NT);
          TB::zero_tail(buf + TA::BYTES, kv, kend, tid, NT);
        }
      }
      block_sync_lds();                  // stage kt is whole, and every wave is done with stage kt - 1
      if (!LAST && kt + STAGES - 1 < nk) issue(kt + STAGES - 1);
      if constexpr (LIVE) {
#pragma unroll
        for (int q = 0; q < BK / 8; ++q) {
          if (GM == GROUP_K && LAST && 8 * q >= kv) break;
          f32x4_t fa[TM], fb[TN];
#pragma unroll
          for (int j = 0; j < TM; ++j) {
            if constexpr (A_T) fa[j] = frag_f32<true, TA>(buf, q, 0, a_nc[j]);
            else fa[j] = frag_f32<false, TA>(buf, q, (wm * TM + j) * 32, kc_off[q]);
          }
#pragma unroll
          for (int i = 0; i < TN; ++i) {
            if constexpr (B_T) fb[i] = frag_f32<true, TB>(buf + TA::BYTES, q, 0, b_nc[i]);
            else fb[i] = frag_f32<false, TB>(buf + TA::BYTES, q, (wn * TN + i) * 32, kc_off[q]);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
              for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[i][r], fa[j][r], acc[i][j], 0, 0, 0);
        }
      }
    };
    auto tile = [&](auto LIVEc) {
      for (int kt = 0; kt + 1 < nk; ++kt) stage(kt, std::false_type{}, LIVEc);
      stage(nk - 1, std::true_type{}, LIVEc);
    };
    if (wm * TM * 32 < mvalid) tile(std::true_type{});
    else tile(std::false_type{});

    // lane (row l32, half lhi) holds columns 8 g + 4 lhi .. + 3 of each 32-column block
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int ml = (wm * TM + j) * 32 + l32;
      if (ml >= mvalid) continue;
      int64_t crow;
      if constexpr (GM == GROUP_M) crow = (int64_t)(off + m0 + ml) * p.ldc;
      else crow = (int64_t)e * p.c_gstride + (int64_t)(m0 + ml) * p.ldc;
#pragma unroll
      for (int i = 0; i < TN; ++i) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int nl = (wn * TN + i) * 32 + 8 * g + 4 * lhi;
          if (nl >= nvalid) continue;
          const int n = n0 + nl;
          float* cp = reinterpret_cast<float*>(p.C) + crow + n;
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * g + r];
          if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_ACT) {
            const float* bp = p.bias + (int64_t)e * p.bias_gstride + n;   // 4-byte aligned only
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] += bp[r];
          }
          if constexpr (EPI == EPI_DACT) {
            const float4 h = *reinterpret_cast<const float4*>(p.aux + crow + n);
            v[0] *= act_bwd(h.x, p.act); v[1] *= act_bwd(h.y, p.act);
            v[2] *= act_bwd(h.z, p.act); v[3] *= act_bwd(h.w, p.act);
          }
          if constexpr (EPI == EPI_SGD) {
            const float4 w = *reinterpret_cast<const float4*>(cp);
            v[0] = w.x - p.lr * v[0]; v[1] = w.y - p.lr * v[1];
            v[2] = w.z - p.lr * v[2]; v[3] = w.w - p.lr * v[3];
          }
          *reinterpret_cast<float4*>(cp) = make_float4(v[0], v[1], v[2], v[3]);
          if constexpr (EPI == EPI_BIAS_ACT)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C2) + crow + n) =
                make_float4(act_fwd(v[0], p.act), act_fwd(v[1], p.act), act_fwd(v[2], p.act), act_fwd(v[3], p.act));
        }
      }
    }
  }
}

template <int BM, int BN, int STAGES>
constexpr size_t gemm_f32_lds_bytes() {
  return (size_t)STAGES * (BM + BN) * F32_BK * 4;
}

}  // namespace dmoe
