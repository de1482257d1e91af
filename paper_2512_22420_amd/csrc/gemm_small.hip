// GEMMs of small windows (a decode step, a draft position: up to 32 rows):
// y = x . w^T with K split over the waves of a workgroup.
//
// At a handful of rows a layer's GEMMs read a few to a few tens of MB, so the
// time is not the weight stream (6.5 TB/s) but what surrounds it.  The
// weight-streaming kernel (gemm.hip) gives a workgroup 128 weight rows and
// fills the chip by splitting K over workgroups, whose partial sums then cross
// memory: stores acknowledged, a counter, a wait, loads -- several microseconds
// per GEMM, more than the stream itself on a small model, and still few
// workgroups where N is small (a 2048 x 2048 projection ran on 32).  Here a
// workgroup owns 16 output columns (one 16-row weight tile; two for SwiGLU's
// gate and up rows and for the two rotated halves of a head) and its waves
// split K: every wave streams its own k-steps of the tile and of x straight
// from memory into MFMA fragments (nothing is shared, so no LDS and no barrier
// in the loop), the waves' sums meet in LDS in wave order, and the epilogue
// follows.  No partials, no counters, and one memory latency where a wave's
// whole share fits in its registers: the 2048 x 2048 projection at 8 rows
// 10.4 -> 4.8 us (8.4 MB; an empty launch takes about 2.5); gemm.hip's small_wins
// has the other shapes and where the streaming kernel stays ahead.
//
// Fragments as in gemm.hip: the packed weight tile of a k-step is the 1 KB that
// the 64 lanes load (lane l: row l & 15, k (l >> 4) * 8 .. + 7), x lanes read
// 16 bytes of row l & 15; results: lane l has weight rows 4 (l >> 4) + i of x
// row l & 15.
#include <algorithm>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace nj {
namespace {

constexpr int kSU = 2;    // k-steps per stage

__device__ __forceinline__ float silu_mul(float gte, float up) { return gte / (1.0f + expf(-gte)) * up; }

struct SmallK {
  const bf16_t* X;
  const bf16_t* W;  // packed
  void* Y;
  int M, Nout, K, KS;
  int xkb, ykb, xg_kb;  // x, the SwiGLU output, the next norm's input k-blocked: [K/32][M][32]
  // RMSNorm folded in, as in gemm.hip; the sums of squares this kernel writes
  // cover 16 columns each (its own tile)
  const float* ssq_in;
  int nt_in;
  float eps;
  const bf16_t* gain;
  bf16_t* xg;
  float* ssq_out;
  int nt_out;
  QkvRope rope;
};

template <int MT, int NW, int EPI>
__global__ __launch_bounds__(NW * 64, 4) void gemm_small_kernel(SmallK a) {  // 128 registers: two workgroups of 8 waves per CU
  constexpr int NT = EPI == kEpiSwiglu || EPI == kEpiQkvRope ? 2 : 1;
  constexpr int kSets = NT + MT <= 3 ? 4 : 2;  // stages in flight per wave
  constexpr int ROWS = MT * 16, NTH = NW * 64;
  __shared__ __attribute__((aligned(16))) f32x4 red[NW][NT * MT][64];
  __shared__ float s_rinv[ROWS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int M = a.M, Nout = a.Nout, K = a.K, KS = a.KS;
  // the workgroup's weight tiles: the tile (residual), gate and up rows
  // (SwiGLU), or 16 dims of a head and the 16 dims they rotate with
  int tile[NT];
  if constexpr (EPI == kEpiSwiglu) {
    tile[0] = blockIdx.x;
    tile[NT - 1] = Nout / 16 + blockIdx.x;
  } else if constexpr (EPI == kEpiQkvRope) {
    tile[0] = (blockIdx.x >> 2) * 8 + (blockIdx.x & 3);
    tile[NT - 1] = tile[0] + 4;
  } else {
    tile[0] = blockIdx.x;
  }
  const int ks0 = wave * KS / NW, nks = (wave + 1) * KS / NW - ks0;  // this wave's k-steps
  const int nst = (nks + kSU - 1) / kSU;

  // Sums of squares of this thread's row first (used after the stream).
  constexpr int LPR = NTH / ROWS >= 32 ? 32 : NTH / ROWS >= 16 ? 16 : 8;  // lanes per row
  constexpr int SQ = kMaxSsqSegments / LPR;
  const bool scaled = EPI != kEpiResidual && EPI != kEpiResidualNorm && a.ssq_in != nullptr;
  float ssq_v[SQ];
  if (scaled) {
    const int row = min((int)threadIdx.x / LPR, ROWS - 1), c = threadIdx.x % LPR;
    const float* sp = a.ssq_in + (size_t)min(row, M - 1) * a.nt_in;
#pragma unroll
    for (int j = 0; j < SQ; ++j) ssq_v[j] = c + LPR * j < a.nt_in ? sp[c + LPR * j] : 0.f;
  }

  const bf16_t* wp[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) wp[t] = a.W + (((size_t)(tile[t] >> 3) * KS + ks0) * 8 + (tile[t] & 7)) * 512 + lane * 8;
  const bf16_t* xp[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const size_t row = min(mt * 16 + r, M - 1);
    xp[mt] = a.X + (a.xkb ? ((size_t)ks0 * M + row) * 32 : row * K + (size_t)ks0 * 32) + g * 8;
  }
  const uint32_t xstep = a.xkb ? M * 32 : 32;  // elements from one k-step to the next

  bf16x8 wf[kSets][kSU][NT], xf[kSets][kSU][MT];
  auto load = [&](auto setc, int st) {
    constexpr int set = decltype(setc)::value;
#pragma unroll
    for (int u = 0; u < kSU; ++u) {
      const int ks = min(st * kSU + u, nks - 1);  // a ragged last stage repeats the last k-step (not multiplied)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        xf[set][u][mt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xp[mt] + ks * xstep));
#pragma unroll
      for (int t = 0; t < NT; ++t)
        wf[set][u][t] = __builtin_bit_cast(
            bf16x8, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wp[t] + (size_t)ks * 4096)));
    }
  };
  f32x4 acc[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[t][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](auto setc, int st) {
    constexpr int set = decltype(setc)::value;
#pragma unroll
    for (int u = 0; u < kSU; ++u)
      if (st * kSU + u < nks)  // uniform
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[set][u][t], xf[set][u][mt], acc[t][mt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // the loads that take over the set stay behind
  };
  // Stage st sits in set st % kSets.  The steady loop issues every load
  // unconditionally (the compiler can then wait for exactly the stage it needs);
  // the last stages run behind it.
  [&]<int... S>(std::integer_sequence<int, S...>) {
    if (nst >= kSets) {
      (load(std::integral_constant<int, S>{}, S), ...);
      __builtin_amdgcn_sched_barrier(0);
      int st = 0;
      for (; st + 2 * kSets <= nst; st += kSets)
        ((compute(std::integral_constant<int, S>{}, st + S), load(std::integral_constant<int, S>{}, st + S + kSets),
          __builtin_amdgcn_sched_barrier(0)), ...);
      ([&] {
        compute(std::integral_constant<int, S>{}, st + S);
        if (st + S + kSets < nst) load(std::integral_constant<int, S>{}, st + S + kSets);
      }(), ...);
      st += kSets;
      ((st + S < nst ? compute(std::integral_constant<int, S>{}, st + S) : (void)0), ...);
    } else {
      ((S < nst ? load(std::integral_constant<int, S>{}, S) : (void)0), ...);
      ((S < nst ? compute(std::integral_constant<int, S>{}, S) : (void)0), ...);
    }
  }(std::make_integer_sequence<int, kSets>{});

#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[wave][t * MT + mt][lane] = acc[t][mt];
  if (scaled) {  // 1/rms of every row: lane sums in order, then a butterfly over the row's lanes
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < SQ; ++j) s += ssq_v[j];
#pragma unroll
    for (int o = 1; o < LPR; o <<= 1) s += __shfl_xor(s, o);
    if (threadIdx.x % LPR == 0 && (int)threadIdx.x / LPR < ROWS) s_rinv[threadIdx.x / LPR] = 1.0f / sqrtf(s / (float)K + a.eps);
  }
  __syncthreads();
  // sum of fragment (t, mt), in wave order, with the row scale
  auto total = [&](int t, int mt) {
    f32x4 v = red[0][t * MT + mt][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][t * MT + mt][lane];
    if (scaled) v *= s_rinv[mt * 16 + r];
    return v;
  };

  if constexpr (EPI == kEpiQkvRope) {
    const QkvRope& rp = a.rope;
    const int hd = blockIdx.x >> 2, j0 = (blockIdx.x & 3) * 16, T = rp.T, H = rp.H, Hkv = rp.Hkv, B = M / T;
    if (hd < H + Hkv) {
      // wave mt rotates row tile mt: lane dims j0 + 4 g .. + 3 and the same + 64
      for (int mt = wave; mt < MT; mt += NW) {
        const f32x4 x1 = total(0, mt), x2 = total(NT - 1, mt);
        const int m = mt * 16 + r;
        if (m < M) {
          const int b = m / T, i = m % T, j = j0 + 4 * g;
          const f32x4* cp = reinterpret_cast<const f32x4*>(rp.cs + ((size_t)m * 64 + j) * 2);  // (cos, sin) pairs
          const f32x4 c0 = cp[0], c1 = cp[1];
          const float cs[4] = {c0[0], c0[2], c1[0], c1[2]}, sn[4] = {c0[1], c0[3], c1[1], c1[3]};
          float lo[4], hi[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            lo[e] = x1[e] * cs[e] - x2[e] * sn[e];
            hi[e] = x2[e] * cs[e] + x1[e] * sn[e];
          }
          bf16_t* dst = (hd < H ? static_cast<bf16_t*>(rp.q_out) + ((size_t)m * H + hd) * 128
                                : static_cast<bf16_t*>(rp.win_k) + (((size_t)b * Hkv + (hd - H)) * kBlock + i) * 128) + j;
          *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3])};
          *reinterpret_cast<u32x2*>(dst + 64) = u32x2{pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
        }
      }
      // unused slots T..15 of the K window blocks: this workgroup's two runs of 16 dims
      if (hd >= H)
        for (int u = threadIdx.x; u < B * (kBlock - T) * 4; u += NTH) {
          const int q = u & 3, s = (u >> 2) % (kBlock - T), b = (u >> 2) / (kBlock - T);
          bf16_t* z = static_cast<bf16_t*>(rp.win_k) + (((size_t)b * Hkv + (hd - H)) * kBlock + T + s) * 128 + j0 + (q >> 1) * 64 + (q & 1) * 8;
          *reinterpret_cast<u32x4*>(z) = u32x4{0u, 0u, 0u, 0u};
        }
    } else {
      // V: one thread per (sequence, head dim) writes the dim's whole 16-slot
      // window row (its T values, then zeros)
      __shared__ float sv[ROWS][33];
      for (int f = wave; f < NT * MT; f += NW) {
        const int t = f / MT, mt = f % MT;
        const f32x4 v = total(t, mt);
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[mt * 16 + r][t * 16 + 4 * g + e] = v[e];
      }
      __syncthreads();
      for (int u = threadIdx.x; u < B * 32; u += NTH) {
        const int b = u >> 5, c = u & 31, dd = j0 + (c & 15) + (c >> 4) * 64;
        uint32_t w[8];
#pragma unroll
        for (int p = 0; p < 8; ++p)
          w[p] = pack_bf16x2(2 * p < T ? sv[b * T + 2 * p][c] : 0.f, 2 * p + 1 < T ? sv[b * T + 2 * p + 1][c] : 0.f);
        u32x4* dst = reinterpret_cast<u32x4*>(static_cast<bf16_t*>(rp.win_v) + (((size_t)b * Hkv + (hd - H - Hkv)) * 128 + dd) * kBlock);
        dst[0] = u32x4{w[0], w[1], w[2], w[3]};
        dst[1] = u32x4{w[4], w[5], w[6], w[7]};
      }
    }
    if (blockIdx.x == 0) {
      for (int u = threadIdx.x; u < B; u += NTH)
        if (rp.ctx_snap) rp.ctx_snap[u] = rp.ctx[u];
      for (int u = threadIdx.x; u < B * Hkv; u += NTH)
        if (rp.attn_cnt) rp.attn_cnt[u * kCounterStride] = 0;
    }
  } else {
    const int n = tile[0] * 16 + 4 * g;
    auto out_at = [&](int kb, int m) { return kb ? ((size_t)(n >> 5) * M + m) * 32 + (n & 31) : (size_t)m * Nout + n; };
    for (int mt = wave; mt < MT; mt += NW) {
      const int m = mt * 16 + r;
      if constexpr (EPI == kEpiSwiglu) {
        const f32x4 gt = total(0, mt), up = total(NT - 1, mt);
        if (m < M)
          *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(a.Y) + out_at(a.ykb, m)) =
              u32x2{pack_bf16x2(silu_mul(gt[0], up[0]), silu_mul(gt[1], up[1])),
                    pack_bf16x2(silu_mul(gt[2], up[2]), silu_mul(gt[3], up[3]))};
      } else {
        const f32x4 v = total(0, mt);
        f32x4* hp = reinterpret_cast<f32x4*>(static_cast<float*>(a.Y) + (size_t)min(m, M - 1) * Nout + n);
        const f32x4 hv = *hp + v;
        if (m < M) *hp = hv;
        if constexpr (EPI == kEpiResidualNorm) {
          const u32x2 gw = *reinterpret_cast<const u32x2*>(a.gain + n);
          if (m < M)
            *reinterpret_cast<u32x2*>(a.xg + out_at(a.xg_kb, m)) =
                u32x2{pack_bf16x2(hv[0] * bf2f((bf16_t)(gw[0] & 0xffffu)), hv[1] * bf2f((bf16_t)(gw[0] >> 16))),
                      pack_bf16x2(hv[2] * bf2f((bf16_t)(gw[1] & 0xffffu)), hv[3] * bf2f((bf16_t)(gw[1] >> 16)))};
          float p = hv[0] * hv[0];
          p = fmaf(hv[1], hv[1], p);
          p = fmaf(hv[2], hv[2], p);
          p = fmaf(hv[3], hv[3], p);
          p += __shfl_xor(p, 16);
          p += __shfl_xor(p, 32);
          if (g == 0 && m < M) a.ssq_out[(size_t)m * a.nt_out + tile[0]] = p;
        }
      }
    }
  }
}

template <int MT, int NW, int EPI>
hipError_t launch_one(const SmallK& a, hipStream_t s) {
  hipLaunchKernelGGL((gemm_small_kernel<MT, NW, EPI>), dim3(a.Nout / (EPI == kEpiQkvRope ? 32 : 16)), dim3(NW * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_small(const void* x, const void* w, void* y, int M, int N, int K, int epi, const GemmPlan& p,
                             const GemmNorm* nm, const QkvRope* rope, hipStream_t s, bool x_kblocked, bool y_kblocked) {
  const int Nout = epi == kEpiSwiglu ? N / 2 : N;
  if (M < 1 || M > 16 * p.mt || p.mt > kSmallMaxTiles || K % 32 || Nout % (epi == kEpiQkvRope ? 128 : 16) ||
      (epi == kEpiQkvRope && !rope) ||
      (y_kblocked && (epi != kEpiSwiglu || Nout % 32)))
    return hipErrorInvalidValue;
  SmallK a{static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w), y, M, Nout, K, K / 32,
           x_kblocked ? 1 : 0, y_kblocked ? 1 : 0, 0, nullptr, 0, 0.f, nullptr, nullptr, nullptr, 0, rope ? *rope : QkvRope{}};
  if (nm) {
    if (nm->ssq_in && (nm->nt_in < 1 || nm->nt_in > kMaxSsqSegments)) return hipErrorInvalidValue;
    a.ssq_in = nm->ssq_in, a.nt_in = nm->nt_in, a.eps = nm->eps;
    if (epi == kEpiResidualNorm) {
      if (!nm->gain || !nm->xg || !nm->ssq_out || (nm->xg_kb && Nout % 32)) return hipErrorInvalidValue;
      a.xg_kb = nm->xg_kb;
      a.gain = static_cast<const bf16_t*>(nm->gain), a.xg = static_cast<bf16_t*>(nm->xg), a.ssq_out = nm->ssq_out;
      a.nt_out = Nout / 16;
    }
  }
  // the forms that gemm_plan picks
  const bool wide = p.nw == 16;
  switch (epi) {
    case kEpiResidual:
      if (p.mt == 1) return launch_one<1, 8, kEpiResidual>(a, s);
      break;
    case kEpiSwiglu:
      if (p.mt == 1) return launch_one<1, 8, kEpiSwiglu>(a, s);
      break;
    case kEpiResidualNorm:
      if (p.mt == 1) return launch_one<1, 8, kEpiResidualNorm>(a, s);
      if (p.mt == 2) return launch_one<2, 8, kEpiResidualNorm>(a, s);
      break;
    case kEpiQkvRope:
      if (p.mt == 1) return wide ? launch_one<1, 16, kEpiQkvRope>(a, s) : launch_one<1, 8, kEpiQkvRope>(a, s);
      if (p.mt == 2) return wide ? launch_one<2, 16, kEpiQkvRope>(a, s) : launch_one<2, 8, kEpiQkvRope>(a, s);
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace nj
