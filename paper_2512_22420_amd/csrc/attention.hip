// Paged verify attention: each sequence's k+1 window queries attend to its
// cached tokens (reached through the block table, 16 tokens per block) and
// causally to the window itself.
//
// bf16 path.  One workgroup (4 waves) per (sequence, KV head, KV split).  The
// G query heads sharing a KV head and the T = k+1 window positions are packed
// into R = T*G query rows (at most 64 = 4 tiles of 16), so every key and value
// byte read from HBM serves all of them.  Blocks are taken in pairs of 32
// tokens: a wave computes
//   S^T (32 tokens x 16 rows) = K . Q^T      with 8 x mfma 16x16x32 bf16,
// the tokens dealt to the MFMAs' rows so that each lane ends up with eight
// consecutive tokens of one query row -- exactly the B operand of
//   O^T (16 dims x 16 rows) += V^T . P^T     with mfma 16x16x32 bf16,
// so the softmax numerators go straight from the score registers into the
// second product with no data exchange.  The A operand V^T needs the same
// eight tokens of one dim: V pages are stored dim-major inside a block
// ([D][16]), which makes that one 16-byte read.  Softmax is online in the log2
// domain.  When the grid splits the KV range, each split writes its partial
// (o, max, sum) and the last split to arrive merges them in split order.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "attn_work.h"
#include "common.h"
#include "kernels.h"

namespace nj {
namespace {

constexpr int kD = 128;  // head dim of the bf16 path
constexpr size_t kStreamBytes = (size_t)128 << 20;
constexpr int kAttnWgsPerCu = 2;  // resident attention workgroups per CU (registers, LDS of the larger forms)

__device__ __forceinline__ bf16x8 ld8(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}

struct AttnK {
  const bf16_t* q;
  const bf16_t* kp;
  const bf16_t* vp;
  const bf16_t* wk;
  const bf16_t* wv;
  const int32_t* table;
  const int32_t* ctx;
  float* part_o;
  float* part_ml;
  int* counters;  // [B*Hkv][kCounterStride] split arrivals, zero on entry (cleared before each launch)
  const AttnWork* work;  // [gridDim.x] the work list (attn_work.h)
  bf16_t* out;
  int* err;
  int max_blocks, num_blocks, T, H, Hkv;
  float scale_log2;
  int part_o_bytes, part_ml_bytes;
  int okbM;  // nonzero: out stored k-blocked, [H*kD/32][okbM][32] (okbM = B*T rows)
};

// output row m = b*T + i, column c = head * kD + d (4 consecutive columns)
__device__ __forceinline__ u32x2* out_at(const AttnK& a, int m, int c) {
  return reinterpret_cast<u32x2*>(a.okbM ? a.out + ((size_t)(c >> 5) * a.okbM + m) * 32 + (c & 31)
                                         : a.out + (size_t)m * a.H * kD + c);
}

// Weight of a partial (o, max m, sum) relative to the max mx of all of them.
// m = -inf: no finite or infinite score, so (o, sum) are zeros, or NaN where
// every score was NaN (the max drops NaN): weighted 0 and still added, which
// keeps the NaN.
__device__ __forceinline__ float rel_weight(float m, float mx) { return m == -INFINITY ? 0.f : exp2f(m - mx); }

// A split has written its partial (o, max, sum) with device-coherent stores;
// count it in, and let the last split of the (sequence, KV head) to arrive
// merge all splits in split order:
//   out = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s.
// A thread merges up to kMergeUnits units of 4 head dims of one query row; the
// (m, l) and o of kMergeSplits splits of all its units are loaded together
// (one memory round trip; reading every (m, l) first cost a second one), and
// more splits than that fold in with a running max.
constexpr int kMergeSplits = 4;
constexpr int kMergeUnits = 4;
__device__ void split_arrive(const AttnK& a, int pair, int nsplit, int slot0, int R, int RT, int G, int b, int kvh,
                             __amdgpu_buffer_rsrc_t ors, __amdgpu_buffer_rsrc_t mrs) {
  __shared__ int s_last;
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    s_last = (__hip_atomic_fetch_add(a.counters + pair * kCounterStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nsplit - 1);
  __syncthreads();
  if (!s_last) return;
  const int rpad = RT * 16;
  const size_t pbase = (size_t)slot0 * rpad;
  const int nunits = R * (kD / 4);
  for (int ub = 0; ub < nunits; ub += 256 * kMergeUnits) {
    f32x4 acc[kMergeUnits];
    float mx[kMergeUnits], wsum[kMergeUnits];
#pragma unroll
    for (int q = 0; q < kMergeUnits; ++q) {
      acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      mx[q] = -INFINITY;
      wsum[q] = 0.f;
    }
    for (int s0 = 0; s0 < nsplit; s0 += kMergeSplits) {
      f32x4 ov[kMergeUnits][kMergeSplits];
      float2 ml[kMergeUnits][kMergeSplits];
#pragma unroll
      for (int q = 0; q < kMergeUnits; ++q) {
        if (ub + q * 256 >= nunits) break;  // uniform
        const int u = min(ub + (int)threadIdx.x + q * 256, nunits - 1);
        const int qr = u / (kD / 4), d = (u % (kD / 4)) * 4;
#pragma unroll
        for (int j = 0; j < kMergeSplits; ++j) {
          const size_t row = pbase + (size_t)min(s0 + j, nsplit - 1) * rpad + qr;
          ml[q][j] = coherent_load_f32x2(mrs, (uint32_t)(row * 8));
          ov[q][j] = coherent_load(ors, (uint32_t)((row * kD + d) * 4));
        }
      }
#pragma unroll
      for (int q = 0; q < kMergeUnits; ++q) {
        if (ub + q * 256 >= nunits) break;
        float bm = -INFINITY;
#pragma unroll
        for (int j = 0; j < kMergeSplits; ++j)
          if (s0 + j < nsplit) bm = fmaxf(bm, ml[q][j].x);
        const float mn = fmaxf(mx[q], bm);
        const float alpha = rel_weight(mx[q], mn);
        acc[q] *= alpha;
        wsum[q] *= alpha;
        mx[q] = mn;
#pragma unroll
        for (int j = 0; j < kMergeSplits; ++j)
          if (s0 + j < nsplit) {
            const float f = rel_weight(ml[q][j].x, mn);
            wsum[q] += f * ml[q][j].y;
            acc[q] += f * ov[q][j];
          }
      }
    }
#pragma unroll
    for (int q = 0; q < kMergeUnits; ++q) {
      const int u = ub + (int)threadIdx.x + q * 256;
      if (u >= nunits) break;
      const int qr = u / (kD / 4), d = (u % (kD / 4)) * 4;
      const float inv = 1.0f / wsum[q];
      const int i = qr / G, hh = qr % G;
      u32x2 o;
      o[0] = pack_bf16x2(acc[q][0] * inv, acc[q][1] * inv);
      o[1] = pack_bf16x2(acc[q][2] * inv, acc[q][3] * inv);
      *out_at(a, b * a.T + i, (kvh * G + hh) * kD + d) = o;
    }
  }
}

// Max over the lanes that share lane % 16 (a query row's four lanes).
__device__ __forceinline__ float row_max(float v) {
  const uint32_t x = __float_as_uint(v);
  const auto p16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const float m = fmaxf(__uint_as_float(p16[0]), __uint_as_float(p16[1]));
  const uint32_t y = __float_as_uint(m);
  const auto p32 = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return fmaxf(__uint_as_float(p32[0]), __uint_as_float(p32[1]));
}

// One online-softmax step of a query row tile: st are this lane's eight scores
// of its row (q . k, -inf where masked); updates the row's reference m_run (log2
// domain: score * scale) and sum and returns the probabilities, relative to
// 2^m_run, as the B operand of the second product.  The reference is the row's
// max, so the token that leads a peaked row has a probability of exactly 1 in
// bf16; a reference that lags the max saves rescales (7B shape, 256 sequences:
// 247 us against 250, nothing at the other shapes) but rounds that token too
// (8B step of 61 sequences: error of the logits 0.0055 against 0.0053).  The accumulators are
// rescaled under a uniform branch, only when a row's max rose.
__device__ __forceinline__ bf16x8 softmax_step(const float (&st)[8], float scale, float& m_run, float& l_run, f32x4 (&o)[8]) {
  float bm = fmaxf(fmaxf(fmaxf(st[0], st[1]), fmaxf(st[2], st[3])), fmaxf(fmaxf(st[4], st[5]), fmaxf(st[6], st[7])));
  bm = row_max(bm) * scale;
  const bool rises = bm > m_run;  // the first valid score does: m_run starts at -inf
  if (__builtin_amdgcn_ballot_w64(rises)) {
    const float mn = rises ? bm : m_run;
    const float alpha = rises ? __builtin_amdgcn_exp2f(m_run - mn) : 1.f;
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt] *= alpha;
    m_run = mn;
  }
  // the hardware exp2 (v_exp_f32) gives exp2(-inf) = 0 for masked tokens; a
  // row with nothing valid yet (m_run = -inf) keeps p = 0
  const float ms = m_run == -INFINITY ? 0.f : m_run;
  float p[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(st[e], scale, -ms));
  l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  u32x4 pp;
#pragma unroll
  for (int e = 0; e < 4; ++e) pp[e] = pack_bf16x2(p[2 * e], p[2 * e + 1]);
  return __builtin_bit_cast(bf16x8, pp);
}

typedef const __attribute__((address_space(1))) char* gptr;
template <bool STREAM>
__device__ __forceinline__ bf16x8 gld8(gptr p) {
  const auto q = reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(p);
  return __builtin_bit_cast(bf16x8, STREAM ? __builtin_nontemporal_load(q) : *q);
}

// Up to 32 query rows (RT = 1 or 2 row tiles).  Each wave takes its own pairs
// of blocks (pair w, w + 4, ... of the split's; split 0 adds the window block
// as a last pair of one) for all the rows, straight from memory into MFMA
// fragments: with one or two row tiles nothing is gained by sharing a block
// through LDS, and without it the loop has no barriers and no LDS reads.  The
// loads in flight set the rate (16 to 32 KB per wave, two waves per SIMD); at
// few blocks per split the chain of dependent accesses (item, page ids,
// blocks, merge) does.  Against the LDS kernel of four-block chunks with
// masks and exec changes in its inner loop (cacheable loads): 8 sequences of
// 1024 tokens at 24 rows 17.5 -> 13.8 us and at 2 rows (8 KV heads) 15.7 -> 13.3
// us, 64 sequences of ~870 tokens at 20 rows 54.7 -> 50.5 us.
//
// A pair is 32 tokens: MFMA h of the score product takes, as row r of its A
// operand, token 8 ((r >> 2) & 1) + 4 h + (r & 3) of block r >> 3, so the lane
// group g = lane / 16 ends up with the scores of tokens 8 (g & 1) .. + 7 of
// block g >> 1 (four from each h): its eight probabilities are the B operand
// of a 16x16x32 MFMA whose A operand is eight consecutive tokens of one dim of
// a V block, one 16-byte load.
constexpr int kRegRow = kD + 4;  // LDS row stride of the wave merge, in floats
template <int RT, bool STREAM>
__global__ __launch_bounds__(256, 2) void attn_reg_kernel(AttnK a) {
  static_assert(RT == 1 || RT == 2, "one or two row tiles");
  constexpr int NP = 4;  // waves
  __shared__ __attribute__((aligned(16))) float s_o[NP][RT * 16 * kRegRow];
  __shared__ float s_m[NP][RT * 16], s_l[NP][RT * 16];
  const AttnWork item = a.work[blockIdx.x];
  if (item.nsplit == 0) return;  // the list is shorter than the grid
  const int b = item.b, kvh = item.kvh, split = item.split, nsplit = item.nsplit;
  const int G = a.H / a.Hkv, R = a.T * G;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int ctx = item.ctx >= 0 ? item.ctx : ~item.ctx;
  if (item.ctx < 0 && threadIdx.x == 0 && split == 0) flag_error(a.err, kErrContext);
  const int c0 = item.c0, c1 = item.c1;
  const int np = (c1 - c0 + 1) / 2;             // pairs of cached blocks
  const int npw = np + (split == 0 ? 1 : 0);    // and the window
  const int n = npw > wave ? (npw - wave + NP - 1) / NP : 0;  // this wave's

  // Page ids of 32 of the wave's pairs: lane l holds block l & 1 of pair
  // idbase + l / 2.  kNoBlock: the window block's memory is read in its place.
  // Past the split's last block that is masked out, with the pair's tokens past
  // the context; for a bad id (any table entry outside [0, num_blocks) of a
  // block inside the context, -1 included) it is not: the window's keys then
  // count as the block's, and the output is invalid, as kErrBlock says.
  constexpr int kNoBlock = INT_MIN;
  int idv = kNoBlock, idbase = 0;
  bool bad = false;
  auto read_ids = [&](int j0) {
    idbase = j0;
    const int p = wave + NP * (j0 + (lane >> 1)), blk = c0 + 2 * p + (lane & 1);
    int id = p < np && blk < c1 ? a.table[(size_t)b * a.max_blocks + blk] : kNoBlock;
    if (id != kNoBlock && (id < 0 || id >= a.num_blocks)) {
      bad = true;
      id = kNoBlock;
    }
    idv = id;
  };
  read_ids(0);

  bf16x8 qf[RT][4];
  int qpos[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int qc = min(t * 16 + r16, R - 1);  // padding rows repeat the last real row
    const int i = qc / G, hh = qc % G;
    const bf16_t* src = a.q + ((size_t)(b * a.T + i) * a.H + kvh * G + hh) * kD + 8 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[t][s] = ld8(src + 32 * s);
    qpos[t] = i;
  }
  const gptr win_k = (gptr)(a.wk + ((size_t)b * a.Hkv + kvh) * (kBlock * kD));
  const gptr win_v = (gptr)(a.wv + ((size_t)b * a.Hkv + kvh) * (kBlock * kD));
  const uint32_t kofs = (uint32_t)((8 * ((r16 >> 2) & 1) + (r16 & 3)) * kD + 8 * g) * 2u;
  const uint32_t vofs = (uint32_t)(r16 * kBlock + 8 * (g & 1)) * 2u;

  // Fragments of two pairs with one row tile, of one pair with two (their
  // accumulators leave no room for more): the next pair's K then loads under
  // this one's softmax and second product, its V from there on.
  constexpr int NS = RT == 1 ? 2 : 1;
  bf16x8 kf[NS][8], vf[NS][8];
  // this lane's block of pair j in the pages (kp or vp), the window block if it has none
  auto page = [&](const bf16_t* pages, gptr win, int j, bool second) {
    const int ia = __builtin_amdgcn_readlane(idv, 2 * (j - idbase)), ib = __builtin_amdgcn_readlane(idv, 2 * (j - idbase) + 1);
    const gptr pa = ia >= 0 ? (gptr)pages + ((size_t)ia * a.Hkv + kvh) * (kBlock * kD * 2) : win;
    const gptr pb = ib >= 0 ? (gptr)pages + ((size_t)ib * a.Hkv + kvh) * (kBlock * kD * 2) : win;
    return second ? pb : pa;
  };
  auto load_k = [&](auto setc, int j) {
    const gptr kl = page(a.kp, win_k, j, (r16 & 8) != 0) + kofs;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < 4; ++s) kf[decltype(setc)::value % NS][h * 4 + s] = gld8<STREAM>(kl + h * (4 * kD * 2) + s * 64);
  };
  auto load_v = [&](auto setc, int j) {
    const gptr vl = page(a.vp, win_v, j, (g & 2) != 0) + vofs;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) vf[decltype(setc)::value % NS][dt] = gld8<STREAM>(vl + dt * (16 * kBlock * 2));
  };

  float m_run[RT], l_run[RT];
  f32x4 o[RT][8];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Pair j, its fragments in set j % NS.  The loads of the pair that takes over
  // the set go out as soon as it is free (the order is
  // pinned: hoisted loads would need registers of their own), past the wave's
  // last pair too (they read the window block): loads that may or may not
  // have been issued would make the compiler wait for every load in flight.
  auto step = [&](auto setc, int j) {
    constexpr int set = decltype(setc)::value % NS;
    const bool last = j == n - 1;  // this pair may hold fewer than 32 tokens, or be the window's
    int lim[RT];
    if (last) {
      // nv valid tokens among this lane's eight; the window is causal besides.
      // V past the valid tokens may hold anything: zero it.
      const int p = wave + NP * j, blk = c0 + 2 * p + (g >> 1);
      const bool win = p >= np;
      const int v = win ? (g < 2 ? a.T : 0) : (blk < c1 ? min(kBlock, ctx - blk * kBlock) : 0);
      const int nv = v - 8 * (g & 1);
#pragma unroll
      for (int t = 0; t < RT; ++t) lim[t] = win ? min(nv, qpos[t] + 1 - 8 * (g & 1)) : nv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t keep = nv >= 2 * e + 2 ? 0xffffffffu : nv == 2 * e + 1 ? 0xffffu : 0u;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          u32x4 w = __builtin_bit_cast(u32x4, vf[set][dt]);
          w[e] &= keep;
          vf[set][dt] = __builtin_bit_cast(bf16x8, w);
        }
      }
    }
    f32x4 st[RT][2];
#pragma unroll
    for (int t = 0; t < RT; ++t) st[t][0] = st[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          st[t][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[set][h * 4 + s], qf[t][s], st[t][h], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (j + NS - idbase >= 32) read_ids(j + NS);
    load_k(setc, j + NS);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 pf[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      float sc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) sc[e] = st[t][e / 4][e % 4];
      if (last) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sc[e] = e < lim[t] ? sc[e] : -INFINITY;
      }
      pf[t] = softmax_step(sc, a.scale_log2, m_run[t], l_run[t], o[t]);
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int t = 0; t < RT; ++t)
        o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[set][dt], pf[t], o[t][dt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(setc, j + NS);
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  load_k(s0, 0);
  load_v(s0, 0);
  if constexpr (NS == 2) {
    load_k(s1, 1);
    load_v(s1, 1);
  }
  for (int j = 0; j < n; ++j) {
    step(s0, j);
    if constexpr (NS == 2) {
      if (++j >= n) break;
      step(s1, j);
    }
  }
  if (__builtin_amdgcn_ballot_w64(bad) && lane == 0) flag_error(a.err, kErrBlock);

  // merge the waves, then store the rows or this split's partial
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    float ls = l_run[t];
    ls += __shfl_xor(ls, 16);
    ls += __shfl_xor(ls, 32);
    if (g == 0) {
      s_m[wave][t * 16 + r16] = m_run[t];
      s_l[wave][t * 16 + r16] = ls;
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<f32x4*>(&s_o[wave][(t * 16 + r16) * kRegRow + 16 * dt + 4 * g]) = o[t][dt];
  }
  __syncthreads();
  const int slot0 = item.slot0;
  const __amdgpu_buffer_rsrc_t ors = coherent_rsrc(a.part_o, a.part_o_bytes);
  const __amdgpu_buffer_rsrc_t mrs = coherent_rsrc(a.part_ml, a.part_ml_bytes);
  for (int u = threadIdx.x; u < R * (kD / 4); u += 256) {
    const int qr = u / (kD / 4), d = (u % (kD / 4)) * 4;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < NP; ++w) mx = fmaxf(mx, s_m[w][qr]);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    float wsum = 0.f;
#pragma unroll
    for (int w = 0; w < NP; ++w) {
      const float f = rel_weight(s_m[w][qr], mx);
      wsum += f * s_l[w][qr];
      acc += f * *reinterpret_cast<const f32x4*>(&s_o[w][qr * kRegRow + d]);
    }
    if (nsplit == 1) {
      const int i = qr / G, hh = qr % G;
      const float inv = 1.0f / wsum;
      u32x2 ov;
      ov[0] = pack_bf16x2(acc[0] * inv, acc[1] * inv);
      ov[1] = pack_bf16x2(acc[2] * inv, acc[3] * inv);
      *out_at(a, b * a.T + i, (kvh * G + hh) * kD + d) = ov;
    } else {
      const size_t row = ((size_t)slot0 + split) * (RT * 16) + qr;
      coherent_store(ors, (uint32_t)((row * kD + d) * 4), acc);
      if (d == 0) {
        coherent_store_f32(mrs, (uint32_t)(row * 8), mx);
        coherent_store_f32(mrs, (uint32_t)(row * 8 + 4), wsum);
      }
    }
  }
  if (nsplit > 1) split_arrive(a, b * a.Hkv + kvh, nsplit, slot0, R, RT, G, b, kvh, ors, mrs);
}

// 33 to 64 query rows (three or four row tiles, one per wave).  The four waves
// share every block, so the pairs are streamed through LDS (kPairBuf buffers of
// one pair, 16 KB; kPairBuf - 1 pairs in flight, no registers held by them) and
// each wave multiplies every pair by its own row tile, with the token order of
// attn_reg_kernel.  Loads go from memory straight into LDS
// (global_load_lds_dwordx4: lane i's 16 bytes land at byte 16 i of the
// instruction's KB, so each lane fetches the global piece that the swizzled
// layout keeps there); each wave loads one of a pair's four 4 KB pieces (K and
// V of two blocks).  96 KB per CU in flight and ~1000 clocks of work per wave
// and pair: 256 sequences of 2400 tokens at 56 rows 272 -> 241 us (5.2 TB/s)
// against four-block chunks with two chunk buffers and 16x16x16 MFMAs.  One
// wave per SIMD with all four row tiles in registers was slower (392 us: the
// fragments pass through accumulation registers), as was reading the blocks
// from memory once per two row tiles (280 us).
//
// Swizzle, in 16-byte units, so that the 16 lanes of a fragment read's phase
// (one g, all r16) hit 16 different positions of the 256 bytes of LDS banks:
// K row `tok` of block `blk` keeps unit u at u ^ tok ^ 4 blk (the 16 rows of
// one MFMA are 8 tokens of each block, and their tok ^ 4 blk are all
// different); V dim d keeps its two halves swapped when bit 3 of d is set.
constexpr int kPairBuf = 4;
constexpr int kPairBytes = 4 * kBlock * kD * 2;  // K of both blocks, then V of both
template <bool STREAM>
__global__ __launch_bounds__(256, 2) void attn_lds_kernel(AttnK a) {
  __shared__ __attribute__((aligned(16))) char smem[kPairBuf * kPairBytes];
  const AttnWork item = a.work[blockIdx.x];
  if (item.nsplit == 0) return;  // the list is shorter than the grid
  const int b = item.b, kvh = item.kvh, split = item.split, nsplit = item.nsplit;
  const int G = a.H / a.Hkv, R = a.T * G, RT = (R + 15) / 16;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int ctx = item.ctx >= 0 ? item.ctx : ~item.ctx;
  if (item.ctx < 0 && threadIdx.x == 0 && split == 0) flag_error(a.err, kErrContext);
  const int c0 = item.c0, c1 = item.c1;
  const int np = (c1 - c0 + 1) / 2;           // pairs of cached blocks
  const int n = np + (split == 0 ? 1 : 0);    // and the window

  // This wave's piece of a pair: block second of it, K (waves 0, 1) or V (2, 3)
  const int second = wave & 1;
  const bool is_v = wave >= 2;
  // Page ids of its block of 64 pairs, pair idbase + lane.  kNoBlock: the window
  // block's memory is read instead.  Past the split's last block that is masked
  // out; for a bad id (any table entry outside [0, num_blocks) of a block inside
  // the context, -1 included) it is not, and the output is invalid, as kErrBlock
  // says.
  constexpr int kNoBlock = INT_MIN;
  int idv = kNoBlock, idbase = 0;
  bool bad = false;
  auto read_ids = [&](int p0) {
    idbase = p0;
    const int blk = c0 + 2 * (p0 + lane) + second;
    int id = p0 + lane < np && blk < c1 ? a.table[(size_t)b * a.max_blocks + blk] : kNoBlock;
    if (id != kNoBlock && (id < 0 || id >= a.num_blocks)) {
      bad = true;
      id = kNoBlock;
    }
    idv = id;
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): no load of the compiler's is left for the loop to wait for
  };
  uint32_t lofs[4];  // byte offsets in the 4 KB block that this lane's pieces come from
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tok = 4 * i + (lane >> 4), dim = 32 * i + (lane >> 1);
    lofs[i] = is_v ? (uint32_t)(dim * 32 + ((lane & 1) ^ ((dim >> 3) & 1)) * 16)
                   : (uint32_t)(tok * 256 + (((lane & 15) ^ tok ^ (4 * second)) & 15) * 16);
  }
  const bf16_t* win = (is_v ? a.wv : a.wk) + ((size_t)b * a.Hkv + kvh) * (kBlock * kD);
  const bf16_t* pages = is_v ? a.vp : a.kp;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  auto issue = [&](int p) {  // pair p (past the last one: the window block again) into buffer p % kPairBuf
    if (p - idbase >= 64) read_ids(p);
    const int id = __builtin_amdgcn_readlane(idv, p - idbase);
    const bf16_t* src = id >= 0 ? pages + ((size_t)id * a.Hkv + kvh) * (kBlock * kD) : win;
    const uint32_t dst = lds0 + (uint32_t)((p % kPairBuf) * kPairBytes + wave * (kBlock * kD * 2));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(lofs[i]), "s"(src), "s"(dst + i * 1024)
                     : "memory", "m0");
      else
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lofs[i]), "s"(src), "s"(dst + i * 1024)
                     : "memory", "m0");
    }
  };

  bf16x8 qf[4];
  int qpos;
  {
    const int qc = min(wave * 16 + r16, R - 1);  // padding rows repeat the last real row
    const int i = qc / G, hh = qc % G;
    const bf16_t* src = a.q + ((size_t)(b * a.T + i) * a.H + kvh * G + hh) * kD + 8 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = ld8(src + 32 * s);
    qpos = i;
  }
  read_ids(0);  // (waits for the queries too)
#pragma unroll
  for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(qf[s]));
  for (int p = 0; p < kPairBuf - 1; ++p) issue(p);

  // fragment read offsets in a buffer
  uint32_t kofs[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int blk = r16 >> 3, tok = 8 * ((r16 >> 2) & 1) + 4 * h + (r16 & 3);
#pragma unroll
    for (int s = 0; s < 4; ++s)
      kofs[h][s] = (uint32_t)(blk * (kBlock * kD * 2) + tok * 256 + (((4 * s + g) ^ tok ^ (4 * blk)) & 15) * 16);
  }
  const uint32_t vofs = (uint32_t)((2 + (g >> 1)) * (kBlock * kD * 2) + r16 * 32 + (((g & 1) ^ (r16 >> 3)) & 1) * 16);

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < n; ++p) {
    // this wave's piece of pair p has landed once at most the later
    // kPairBuf - 2 pairs' loads are outstanding; after the barrier every
    // wave's has, and every wave is done with pair p - 1, whose buffer takes
    // pair p + kPairBuf - 1
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kPairBuf - 2) * 4) : "memory");
    issue(p + kPairBuf - 1);
    if (wave >= RT) continue;  // uniform
    const char* buf = smem + (p % kPairBuf) * kPairBytes;
    bf16x8 kf[2][4], vf[8];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) kf[h][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + kofs[h][s]));
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) vf[dt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + vofs + dt * 512));
    f32x4 st[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) st[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[h][s], qf[s], st[h], 0, 0, 0);
    float sc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sc[e] = st[e / 4][e % 4];
    if (p >= np - 1) {
      // the last cached pair may hold fewer than 32 tokens; the window is
      // causal.  V past the valid tokens may hold anything: zero it.
      const int blk = c0 + 2 * p + (g >> 1);
      const bool w = p >= np;
      const int v = w ? (g < 2 ? a.T : 0) : (blk < c1 ? min(kBlock, ctx - blk * kBlock) : 0);
      const int nv = v - 8 * (g & 1), lim = w ? min(nv, qpos + 1 - 8 * (g & 1)) : nv;
#pragma unroll
      for (int e = 0; e < 8; ++e) sc[e] = e < lim ? sc[e] : -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t keep = nv >= 2 * e + 2 ? 0xffffffffu : nv == 2 * e + 1 ? 0xffffu : 0u;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
          u32x4 x = __builtin_bit_cast(u32x4, vf[dt]);
          x[e] &= keep;
          vf[dt] = __builtin_bit_cast(bf16x8, x);
        }
      }
    }
    const bf16x8 pf = softmax_step(sc, a.scale_log2, m_run, l_run, o);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pf, o[dt], 0, 0, 0);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the surplus loads, before the workgroup ends
  if (__builtin_amdgcn_ballot_w64(bad) && lane == 0) flag_error(a.err, kErrBlock);

  // every wave holds its rows whole: lane (r16, g) has dims 16 dt + 4 g .. + 3 of row r16
  const int slot0 = item.slot0;
  const __amdgpu_buffer_rsrc_t ors = coherent_rsrc(a.part_o, a.part_o_bytes);
  const __amdgpu_buffer_rsrc_t mrs = coherent_rsrc(a.part_ml, a.part_ml_bytes);
  float lsum = l_run;
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  const int qr = wave * 16 + r16;
  if (qr < R) {
    if (nsplit == 1) {
      const int i = qr / G, hh = qr % G;
      const float inv = 1.0f / lsum;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {
        u32x2 ov;
        ov[0] = pack_bf16x2(o[dt][0] * inv, o[dt][1] * inv);
        ov[1] = pack_bf16x2(o[dt][2] * inv, o[dt][3] * inv);
        *out_at(a, b * a.T + i, (kvh * G + hh) * kD + 16 * dt + 4 * g) = ov;
      }
    } else {
      const size_t row = ((size_t)slot0 + split) * (RT * 16) + qr;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) coherent_store(ors, (uint32_t)((row * kD + 16 * dt + 4 * g) * 4), o[dt]);
      if (g == 0) {
        coherent_store_f32(mrs, (uint32_t)(row * 8), m_run);
        coherent_store_f32(mrs, (uint32_t)(row * 8 + 4), lsum);
      }
    }
  }
  if (nsplit > 1) split_arrive(a, b * a.Hkv + kvh, nsplit, slot0, R, RT, G, b, kvh, ors, mrs);
}

// fp32 path: one workgroup per (sequence, query head, window position); scores
// in LDS, exact softmax, then one thread per output dim.  Short contexts, so
// latency: a thread's K row and its dim's 16 values of a V block come as wide
// loads issued together, and the page ids of 64 blocks are read at once (one
// load per token and id, each waited for, took 21.4 us at two sequences of ~40
// tokens, now 7.9).  Sums keep their order (dims, then tokens, ascending).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // fp32 pages need no 16-byte alignment
struct AttnF {
  const float* q;
  const float* kp;
  const float* vp;
  const float* wk;
  const float* wv;
  const int32_t* table;
  const int32_t* ctx;
  float* out;
  int* err;
  int max_blocks, num_blocks, T, H, Hkv, D;
  float scale;
};

__global__ __launch_bounds__(128) void attn_f32_kernel(AttnF a) {
  extern __shared__ float sc[];
  __shared__ float red[2];
  __shared__ float wred[2];
  const int b = blockIdx.x / a.H, h = blockIdx.x % a.H, i = blockIdx.y;
  const int G = a.H / a.Hkv, kvh = h / G, D = a.D;
  int ctx = a.ctx[b];
  if (ctx < 0 || ctx + a.T > a.max_blocks * kBlock) {
    if (threadIdx.x == 0 && h == 0 && i == 0) flag_error(a.err, kErrContext);
    ctx = max(0, min(ctx, a.max_blocks * kBlock - a.T));
  }
  const int n = ctx + i + 1;
  const float* qr = a.q + ((size_t)(b * a.T + i) * a.H + h) * D;
  float mx = -INFINITY;
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    const float* kr;
    if (t < ctx) {
      const int phys = a.table[(size_t)b * a.max_blocks + t / kBlock];
      if (phys < 0 || phys >= a.num_blocks) {
        flag_error(a.err, kErrBlock);
        sc[t] = -INFINITY;
        continue;
      }
      kr = a.kp + (((size_t)phys * a.Hkv + kvh) * kBlock + t % kBlock) * D;
    } else {
      kr = a.wk + (((size_t)b * a.Hkv + kvh) * kBlock + (t - ctx)) * D;
    }
    float dot = 0.f;
    for (int d0 = 0; d0 < D; d0 += 8) {  // D % 8 == 0
      const f32x4u k0 = *reinterpret_cast<const f32x4u*>(kr + d0), k1 = *reinterpret_cast<const f32x4u*>(kr + d0 + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) dot = fmaf(qr[d0 + e], e < 4 ? k0[e] : k1[e - 4], dot);
    }
    sc[t] = dot * a.scale;
    mx = fmaxf(mx, sc[t]);
  }
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(red[0], red[1]);
  float sum = 0.f;
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    const float e = (sc[t] == -INFINITY) ? 0.f : expf(sc[t] - mx);
    sc[t] = e;
    sum += e;
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((threadIdx.x & 63) == 0) wred[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = wred[0] + wred[1];
  // every lane of a wave walks the same blocks (surplus lanes repeat the last
  // dim), so the page ids are lane reads
  for (int d0 = 0; d0 < D; d0 += blockDim.x) {
    if (d0 + (int)(threadIdx.x & ~63u) >= D) break;  // a whole wave past the last dim
    const int d = min(d0 + (int)threadIdx.x, D - 1);
    float acc = 0.f;
    const int nb = (ctx + kBlock - 1) / kBlock;
    for (int g0 = 0; g0 < nb; g0 += kWave) {
      const int mine = g0 + (threadIdx.x & 63);
      const int ids = mine < nb ? a.table[(size_t)b * a.max_blocks + mine] : -1;
      const int gn = min(kWave, nb - g0);
#pragma unroll 2
      for (int j = 0; j < gn; ++j) {
        const int phys = __builtin_amdgcn_readlane(ids, j);
        if (phys < 0 || phys >= a.num_blocks) continue;
        const float* vr = a.vp + (((size_t)phys * a.Hkv + kvh) * D + d) * kBlock;
        f32x4u v[kBlock / 4];
#pragma unroll
        for (int e = 0; e < kBlock / 4; ++e) v[e] = *reinterpret_cast<const f32x4u*>(vr + 4 * e);
        const int t0 = (g0 + j) * kBlock, nt = min(kBlock, ctx - t0);  // uniform
#pragma unroll
        for (int e = 0; e < kBlock; ++e)
          if (e < nt) acc = fmaf(sc[t0 + e], v[e / 4][e % 4], acc);
      }
    }
    const float* vw = a.wv + (((size_t)b * a.Hkv + kvh) * D + d) * kBlock;
    f32x4u v[kBlock / 4];
#pragma unroll
    for (int e = 0; e < kBlock / 4; ++e) v[e] = *reinterpret_cast<const f32x4u*>(vw + 4 * e);
#pragma unroll
    for (int e = 0; e < kBlock; ++e)
      if (e <= i) acc = fmaf(sc[ctx + e], v[e / 4][e % 4], acc);
    if (d0 + (int)threadIdx.x < D) a.out[((size_t)(b * a.T + i) * a.H + h) * D + d] = acc / sum;
  }
}

}  // namespace

int attention_plan(int B, int Hkv, int max_blocks) {
  // Workgroups of the work list: one per (sequence, KV head) plus up to
  // kExtraWorkgroups more, and no more than the splits of kMinSplitBlocks
  // blocks the longest possible context could use.  The list sizes the
  // splits from the actual context lengths to fit this grid, so a long
  // sequence gets proportionally more splits than a short one.  Once the
  // pairs alone fill half of the resident attention workgroups, fewer extra
  // ones: the grid runs in rounds anyway, and longer splits pay their fixed
  // start-up and merge once per more blocks (measured: 8B B=64 k=4 and the
  // 7B shape at B=256 k=7 fastest with 128 extra, B=8 with 512).
  const int pairs = B * Hkv;
  const long cap = (long)pairs * std::max(1, (max_blocks + kMinSplitBlocks - 1) / kMinSplitBlocks);
  const int extra = 2 * pairs <= kAttnWgsPerCu * device_cus() ? kExtraWorkgroups
                                                                                      : std::min(kExtraWorkgroups, kExtraWorkgroupsLarge);
  return (int)std::max<long>(pairs, std::min<long>((long)pairs + extra, cap));
}

bool attention_orders(int nwg) { return nwg > kAttnWgsPerCu * device_cus(); }

size_t attention_work_bytes(int B, int Hkv) { return (size_t)(B * Hkv + kExtraWorkgroups) * sizeof(AttnWork); }

size_t attention_partial_floats(int B, int Hkv, int T, int G, int D) {
  const int rpad = ((T * G + 15) / 16) * 16;
  return (size_t)(B * Hkv + kExtraWorkgroups) * rpad * (D + 2);
}

namespace {
// One workgroup: the work list of the next attention launches, and (when
// counters is given) their split arrival counters cleared.
__global__ __launch_bounds__(256) void attn_plan_kernel(const int32_t* __restrict__ ctx, int B, int Hkv, int T,
                                                        int max_blocks, int nwg, int order, AttnWork* __restrict__ work,
                                                        int* __restrict__ counters) {
  __shared__ int scratch[attn_work_scratch_ints(256)];
  if (counters)
    for (int u = threadIdx.x; u < B * Hkv; u += 256) counters[u * kCounterStride] = 0;
  build_attn_work<256>(ctx, B, Hkv, T, max_blocks, nwg, order != 0, work, scratch);
}
}  // namespace

hipError_t launch_attn_plan(const int32_t* ctx, int B, int Hkv, int T, int max_blocks, int nwg, void* work,
                            int* counters, hipStream_t s) {
  if (nwg < B * Hkv || nwg > B * Hkv + kExtraWorkgroups) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(256), 0, s, ctx, B, Hkv, T, max_blocks, nwg,
                     attention_orders(nwg) ? 1 : 0, static_cast<AttnWork*>(work), counters);
  return hipGetLastError();
}

hipError_t launch_attention(const AttnArgs& x, hipStream_t s) {
  const int G = x.H / x.Hkv;
  if (x.dtype == kF32) {
    AttnF a{static_cast<const float*>(x.q), static_cast<const float*>(x.k_pages),
            static_cast<const float*>(x.v_pages), static_cast<const float*>(x.win_k),
            static_cast<const float*>(x.win_v), x.block_table, x.ctx, static_cast<float*>(x.out), x.err,
            x.max_blocks, x.num_blocks, x.T, x.H, x.Hkv, x.D, 1.0f / sqrtf((float)x.D)};
    const size_t lds = (size_t)x.max_blocks * kBlock * sizeof(float);
    hipLaunchKernelGGL(attn_f32_kernel, dim3(x.B * x.H, x.T), dim3(128), lds, s, a);
    return hipGetLastError();
  }
  const int R = x.T * G, RT = (R + 15) / 16;
  AttnK a{static_cast<const bf16_t*>(x.q), static_cast<const bf16_t*>(x.k_pages),
          static_cast<const bf16_t*>(x.v_pages), static_cast<const bf16_t*>(x.win_k),
          static_cast<const bf16_t*>(x.win_v), x.block_table, x.ctx, x.part_o, x.part_ml, x.counters,
          x.work, static_cast<bf16_t*>(x.out), x.err, x.max_blocks, x.num_blocks, x.T, x.H, x.Hkv,
          (float)(1.4426950408889634 / sqrt((double)kD)),
          (int)std::min<size_t>(attention_partial_floats(x.B, x.Hkv, x.T, G, kD) / (kD + 2) * kD * 4, INT32_MAX),
          (int)std::min<size_t>(attention_partial_floats(x.B, x.Hkv, x.T, G, kD) / (kD + 2) * 2 * 4, INT32_MAX),
          x.out_kblocked ? x.B * x.T : 0};
  if (!x.work || x.wgs < x.B * x.Hkv || x.wgs > x.B * x.Hkv + kExtraWorkgroups) return hipErrorInvalidValue;
  // A cache read that does not stay in the last-level cache (256 MB) until the
  // layer comes round again goes non-temporal, which reads faster from HBM.
  // Measured with plain -> streaming loads (us; tables as wide as the contexts,
  // caches from HBM): 8B at 250 MB 56.1 -> 51.5, at 190 MB 47.7 -> 46.4, at 130
  // MB 44.0 -> 45.1; 7B with 56 rows at 360 MB 83.0 -> 73.7, at 140 MB 57.4 ->
  // 54.5, at 95 MB 52.3 -> 49.9, at 48 MB 33.5 -> 33.2; 1B at 255 MB 62.1 ->
  // 59.1, at 128 MB 42.3 -> 42.6: the line of 128 MB lies where they cross, by
  // 2-5% earlier or later by shape.  A cache of up to 220 MB that is still in the
  // last-level cache loses up to 15% (8B at 160 MB 38.1 -> 44.0), but a model's
  // other layers and weights come between.  The host knows the contexts that the
  // table allows, not the contexts: in a wider table a small read streams too,
  // which costs up to 5% (32 MB 20.0 -> 20.0, 10 MB 15.9 -> 16.2, 96 MB 38.4 ->
  // 40.1).
  const bool stream = (size_t)x.B * x.max_blocks * x.Hkv * (2 * kBlock * kD * 2) > kStreamBytes;
  const dim3 grid(x.wgs), block(256);
  if (RT == 1) {
    if (stream) hipLaunchKernelGGL((attn_reg_kernel<1, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((attn_reg_kernel<1, false>), grid, block, 0, s, a);
  } else if (RT == 2) {
    if (stream) hipLaunchKernelGGL((attn_reg_kernel<2, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((attn_reg_kernel<2, false>), grid, block, 0, s, a);
  } else {
    if (stream) hipLaunchKernelGGL(attn_lds_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(attn_lds_kernel<false>, grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace nj
