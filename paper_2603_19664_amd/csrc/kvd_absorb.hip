// Value-absorbed fused recompute + attention (AbsorbArgs): kernels and launchers.
//
// The tiled engines spend 4 d head_dim flop per (token, KV head): 2 d head_dim
// on its key and 2 d head_dim on its value.  No single value is needed, only
// their probability-weighted sum, and that is one projection of the weighted
// sum of the normalised residuals.  So the value half of the token GEMM becomes
// a second, streamed read of the residuals (2 n_q d flop per token instead of
// 2 n_kv head_dim d) and one small product per call.  Measured on MI355X, calls
// back to back, both paths in turn (Gemma-3-4B layer shape, packed weights): B = 16
// x 2560 tokens with 100 stored rows 387 -> 265 us, B = 8 x 3072 with 1025 stored
// rows 250 -> 172, B = 1 x 4096 49.3 -> 44.5 (54.8 -> 52.8 with events around each
// call); the two extra launches (about 15 us) are why smaller calls stay on the
// tiled engines.
#include <atomic>

#include "kvd_device.hpp"
#include "kvd_launch.h"

namespace kvd {

// ------------------------------------------------------------------ scores

// Element of the scores of (b, token t, query head h): per 32-token block, the 4
// tokens 8 lg + 4 half .. of every head in one run, so that a wave of the absorb
// kernel reads a block in contiguous pieces (with a row per head its strided
// 16-byte reads took as long as the residuals': 13.1 us at B = 1 x 4096 tokens).
__device__ __forceinline__ size_t score_at(const AbsorbArgs& a, int b, int t, int h) {
  const int e = t & 31;
  return ((size_t)b * a.Tp + (t & ~31)) * a.n_q + (((e & 4) + (e >> 3)) * a.n_q + h) * 4 + (e & 3);
}

// One workgroup: RW rows of W_k (RW / HD heads) for MT tokens on WideTile's
// K-loop (MFMA-bound at large grids: B = 16 x 2560 tokens in 217 us, 1.0 PFLOP/s;
// at B = 1 x 4096 the 40 K-steps of one round, 28 us), then per token the dot product of the rotated
// rows with each query head of the rows' KV head.  The keys stay in fp32
// accumulators and are never stored.
template <class Tile, int HD, int RW, int MT, bool FOLD>
__global__ __launch_bounds__(Tile::NT, 1) void score_kernel(AbsorbArgs a, int per_xcd, int hg) {
  extern __shared__ __align__(16) char lds[];
  constexpr int NT = Tile::NT;
  constexpr int NH = RW / HD;                     // heads per tile
  static_assert(RW % HD == 0, "whole heads");
  constexpr int BPH = HD / 32;                    // 32-row blocks per head
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int C = (a.T + MT - 1) / MT;
  const int n_rg = a.n_kv * HD / RW;
  const unsigned item = (blockIdx.x % kXcds) * (unsigned)per_xcd + blockIdx.x / kXcds;
  const unsigned n_items = (unsigned)n_rg * (unsigned)a.B * (unsigned)C;
  if (item >= n_items) return;
  // the next kernel's arrival counters start at zero whatever the workspace held
  for (size_t i = (size_t)item * NT + tid; i < (size_t)a.n_done; i += (size_t)n_items * NT) a.done[i] = 0u;
  // items as in the fused kernels: groups of hg row groups of one sequence,
  // token tiles in order, row groups alternating
  const int hg_log2 = __builtin_ctz((unsigned)hg);
  const unsigned hgC = (unsigned)C << hg_log2;
  const unsigned gi = item / hgC, rem = item - gi * hgC;
  const int jg = (int)(gi / (unsigned)a.B);
  const int b = (int)(gi - (unsigned)jg * (unsigned)a.B);
  const int t0 = (int)(rem >> hg_log2) * MT;
  const int rg = (jg << hg_log2) + (int)(rem & (unsigned)(hg - 1));
  const int n = min(MT, a.T - t0);
  const int g = a.n_q / a.n_kv;
  const int j0 = rg * NH;
  const ScoreLds L = score_lds(HD, g, RW, MT, a.d);
  double* rev = reinterpret_cast<double*>(lds + L.rev);
  float* rinv = reinterpret_cast<float*>(lds + L.rinv);
  int* pos = reinterpret_cast<int*>(lds + L.pos);
  uint16_t* hst = reinterpret_cast<uint16_t*>(lds + L.hst);
  float* red = reinterpret_cast<float*>(lds + L.hst);
  float* qs = reinterpret_cast<float*>(lds + L.q);
  uint16_t* gam = reinterpret_cast<uint16_t*>(lds + L.gam);
  auto setup = [&]() {
    const int p0 = (a.pos0 != nullptr ? a.pos0[b] : 0) + t0;
    if (tid < MT) pos[tid] = p0 + tid;
    if (tid < HD / 2) rev[tid] = a.rev[tid];
    if constexpr (!FOLD)
      for (int i = tid; i < a.d / 8; i += NT)
        *reinterpret_cast<uint4*>(gam + 8 * i) = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.gamma) + 8 * i);
    const uint16_t* q = static_cast<const uint16_t*>(a.q) + ((size_t)b * a.n_q + (size_t)j0 * g) * HD;
    for (int i = tid; i < NH * g * HD / 8; i += NT) {
      float x[8];
      load8(q + 8 * i, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) qs[8 * i + e] = x[e] * ScoreScale<HD>::v;
    }
  };
  const uint16_t* wk = static_cast<const uint16_t*>(a.w_k) + (size_t)rg * RW * a.d;
  const Half halves[2] = {Half{wk, 1}, Half{Tile::SPLIT ? nullptr : wk + (size_t)(RW / 2) * a.d, 1}};
  Tile::run_with(
      static_cast<const uint16_t*>(a.h) + ((size_t)b * a.h_ld + t0) * a.d, n, gam,
      static_cast<const uint16_t*>(a.gamma), a.d, a.eps, halves, hst, rinv, setup,
      [&](f32x16_t (&acc)[Tile::NB_F][Tile::NB_T], const bool (&)[Tile::NB_F]) {
        // rotate the rows in place, then one dot product per query head
#pragma unroll
        for (int bt = 0; bt < Tile::NB_T; ++bt) {
          const int tok = 32 * bt + (lane & 31);
          const float ri = rinv[tok];
          const int p = pos[tok];
#pragma unroll
          for (int bf = 0; bf < Tile::NB_F; ++bf) {
            int half, row0;
            Tile::block_rows(w, bf, half, row0);
            const int tr = half * (RW / 2) + row0;                     // row in the tile
            const int f0 = tr % HD + 4 * (lane >> 5);   // feature of register 0
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
              float x0 = acc[bf][bt][r] * ri, x1 = acc[bf][bt][r + 1] * ri;
              rope_rotate(x0, x1, p, rev[(f0 + 8 * (r >> 2) + (r & 3)) >> 1]);
              acc[bf][bt][r] = x0;
              acc[bf][bt][r + 1] = x1;
            }
          }
        }
        for (int h0 = 0; h0 < g; h0 += kScoreHeads) {
          const int nh = min(kScoreHeads, g - h0);
          for (int hq = 0; hq < nh; ++hq) {
#pragma unroll
            for (int bf = 0; bf < Tile::NB_F; ++bf) {
              int half, row0;
              Tile::block_rows(w, bf, half, row0);
              const int tr = half * (RW / 2) + row0;
              const int f0 = tr % HD + 4 * (lane >> 5);
              const float* qh = qs + ((size_t)(tr / HD) * g + h0 + hq) * HD + f0;
              float4 qv[4];
#pragma unroll
              for (int k = 0; k < 4; ++k) qv[k] = *reinterpret_cast<const float4*>(qh + 8 * k);
#pragma unroll
              for (int bt = 0; bt < Tile::NB_T; ++bt) {
                float s = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                  s = fmaf(acc[bf][bt][4 * k + 0], qv[k].x, s);
                  s = fmaf(acc[bf][bt][4 * k + 1], qv[k].y, s);
                  s = fmaf(acc[bf][bt][4 * k + 2], qv[k].z, s);
                  s = fmaf(acc[bf][bt][4 * k + 3], qv[k].w, s);
                }
                s += __shfl_xor(s, 32, 64);
                if (lane < 32) red[((size_t)(tr / 32) * kScoreHeads + hq) * MT + 32 * bt + lane] = s;
              }
            }
          }
          __syncthreads();
          for (int i = tid; i < NH * nh * MT; i += NT) {
            const int tok = i % MT, r = i / MT, hq = r % nh, hd = r / nh;
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < BPH; ++k) s += red[((size_t)(hd * BPH + k) * kScoreHeads + hq) * MT + tok];
            a.scores[score_at(a, b, t0 + tok, (j0 + hd) * g + h0 + hq)] = tok < n ? s : -INFINITY;
          }
          __syncthreads();
        }
        if (rg == 0 && tid < MT) a.rinv[(size_t)b * a.Tp + t0 + tid] = rinv[tid];
      });
}

// ------------------------------------------------------------------ probability-weighted residual sums

// Stored-tail tile c of (b, KV head j): as the fused kernels' tail chunks.
template <int HD>
__device__ __forceinline__ void tail_tile(const AbsorbArgs& a, int item, int rows, char* lds) {
  constexpr int NT = 64 * kAbsorbWaves;
  constexpr int KLD = kv_ld<uint16_t>(HD);
  const int c = item % a.n_tail, bj = item / a.n_tail;
  const int j = bj % a.n_kv, b = bj / a.n_kv;
  const int g = a.n_q / a.n_kv;
  const AttnLds AL = attn_lds(align_up(sizeof(uint16_t) * (size_t)rows * KLD, 16), g, HD, rows);
  uint16_t* kv = reinterpret_cast<uint16_t*>(lds);
  const int r0 = c * kTile;
  const int nk = c == a.n_tail - 1 ? a.T_tail - r0 : kTile;
  load_q<uint16_t, HD, NT>(static_cast<const uint16_t*>(a.q), b, a.n_q, j, g, reinterpret_cast<float*>(lds + AL.q));
  int s0 = a.tail_t_off + r0;
  s0 -= s0 >= a.tail_t_cap ? a.tail_t_cap : 0;
  load_kv_tile<uint16_t, HD, NT>(static_cast<const uint16_t*>(a.tk), static_cast<const uint16_t*>(a.tv), b, a.n_kv, j,
                                 a.tail_t_cap, s0, min(nk, kTile), kv);
  if (nk > kTile) {
    s0 += kTile;
    s0 -= s0 >= a.tail_t_cap ? a.tail_t_cap : 0;
    load_kv_tile<uint16_t, HD, NT>(static_cast<const uint16_t*>(a.tk), static_cast<const uint16_t*>(a.tv), b, a.n_kv,
                                   j, a.tail_t_cap, s0, nk - kTile, kv + (size_t)kTile * KLD);
  }
  __syncthreads();
  attend_tile<uint16_t, HD, NT, 2>(kv, nk, rows, g, lds, AL);
  write_partial<HD, NT>(lds, AL, a.tacc, a.tml, b, a.n_q, j, g, a.n_tail, c, 1);
}

// grid: n_tail * n_kv * B tail tiles, then (columns / 128) * S * B ranges.  A wave
// takes 32-token steps of its range (step i to wave i % kAbsorbWaves): p r as MFMA A rows
// (16 query heads x 32 tokens, split into two bf16 parts so that 16 bits of
// mantissa survive; with PACK, at most 8 heads, the low parts are rows 8..15),
// the residual rows as B: 8 rows x 16 bytes per lane, transposed in registers
// by byte permutes (row-major rows in memory, tokens in MFMA k order).
// Bound by the residual stream: 210 MB (B = 16 x 2560 tokens) in 43 us, 4.9 TB/s;
// 4 waves per workgroup so that two share a CU and cover each other's first
// loads and merge (50 us with 8 waves).  At B = 1 (21 MB, 13 us) the launch, the
// first round trip and the ranges' merge are most of it.
template <int HD, bool PACK>
__global__ __launch_bounds__(64 * kAbsorbWaves, 2) void absorb_kernel(AbsorbArgs a, int tail_rows) {
  extern __shared__ __align__(16) char lds[];
  constexpr int NT = 64 * kAbsorbWaves;
  int item = blockIdx.x;
  const int n_tail = a.n_tail * a.n_kv * a.B;
  if (item < n_tail) {
    tail_tile<HD>(a, item, tail_rows, lds);
    return;
  }
  item -= n_tail;
  const int n_sl = (a.d + kAbsorbCols - 1) / kAbsorbCols;
  const int sl = item % n_sl, bs = item / n_sl;
  const int s = bs % a.S, b = bs / a.S;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int lq = lane & 15, lg = lane >> 4;
  // range s: the 32-token blocks s, s + S, ... counted from the last token back
  // (the score kernel's latest rows are the ones a cache still holds)
  const int nb = (a.T + kAbsorbBlock - 1) / kAbsorbBlock;
  const int nblk = (nb - s + a.S - 1) / a.S;
  const int col = min(sl * kAbsorbCols + 8 * lq, a.d - 8);  // d is a multiple of 64: the last slice may be half empty
  const int head = min(PACK ? lq & 7 : lq, a.n_q - 1);
  const float* sp = a.scores + (size_t)b * a.Tp * a.n_q + (lg * a.n_q + head) * 4;
  const float* rp = a.rinv + (size_t)b * a.Tp + 8 * lg;
  const uint16_t* hp = static_cast<const uint16_t*>(a.h) + (size_t)b * a.h_ld * a.d + col;

  f32x4_t acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = {0.0f, 0.0f, 0.0f, 0.0f};
  float m = -INFINITY, l = 0.0f;
  constexpr int D = kAbsorbDepth;
  uint4 hv[D][8];
  float4 sv[D][2], rv[D][2];
  const int steps = (nblk - w + kAbsorbWaves - 1) / kAbsorbWaves;
  auto load = [&](int k, int i) {  // the wave's step i (steps past its last repeat it)
    const int t = kAbsorbBlock * (nb - 1 - ((w + kAbsorbWaves * min(i, steps - 1)) * a.S + s));
    sv[k][0] = *reinterpret_cast<const float4*>(sp + (size_t)t * a.n_q);
    sv[k][1] = *reinterpret_cast<const float4*>(sp + (size_t)t * a.n_q + 16 * a.n_q);
    rv[k][0] = *reinterpret_cast<const float4*>(rp + t);
    rv[k][1] = *reinterpret_cast<const float4*>(rp + t + 4);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      hv[k][j] = *reinterpret_cast<const uint4*>(hp + (size_t)min(t + 8 * lg + j, a.T - 1) * a.d);
  };
  auto step = [&](int k) {
    const float x[8] = {sv[k][0].x, sv[k][0].y, sv[k][0].z, sv[k][0].w, sv[k][1].x, sv[k][1].y, sv[k][1].z, sv[k][1].w};
    const float r[8] = {rv[k][0].x, rv[k][0].y, rv[k][0].z, rv[k][0].w, rv[k][1].x, rv[k][1].y, rv[k][1].z, rv[k][1].w};
    float bm = x[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) bm = fmaxf(bm, x[e]);
    bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
    bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
    if (__any(bm > m)) {  // a new maximum in some head: rescale the running sums
      const float mn = fmaxf(m, bm);
      const float f = exp2f(m - mn);
      m = mn;
      l *= f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float fi = __shfl(f, 4 * lg + i, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e][i] *= fi;
      }
    }
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const float p0 = exp2f(x[e] - m), p1 = exp2f(x[e + 1] - m);
      l += p0 + p1;
      const float w0 = p0 * r[e], w1 = p1 * r[e + 1];
      hi[e / 2] = pack_bf16x2(w0, w1);
      lo[e / 2] = pack_bf16x2(w0 - bf_lo(hi[e / 2]), w1 - bf_hi(hi[e / 2]));
    }
    const bf16x8_t ah = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
    const bf16x8_t al = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    bf16x8_t ap = ah;
    if constexpr (PACK) ap = lq < 8 ? ah : al;
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // dword c of the rows: columns 2 c, 2 c + 1
      uint32_t d[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = c == 0 ? hv[k][j].x : c == 1 ? hv[k][j].y : c == 2 ? hv[k][j].z : hv[k][j].w;
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const uint32_t sel = o ? 0x07060302u : 0x05040100u;
        const bf16x8_t bv = __builtin_bit_cast(
            bf16x8_t, make_uint4(__builtin_amdgcn_perm(d[1], d[0], sel), __builtin_amdgcn_perm(d[3], d[2], sel),
                                 __builtin_amdgcn_perm(d[5], d[4], sel), __builtin_amdgcn_perm(d[7], d[6], sel)));
        acc[2 * c + o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap, bv, acc[2 * c + o], 0, 0, 0);
        if constexpr (!PACK) acc[2 * c + o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bv, acc[2 * c + o], 0, 0, 0);
      }
    }
  };
  // D - 1 steps in flight ahead of the one being added; loads are unconditional
  // so that the waits count them statically
  if (steps > 0) {
#pragma unroll
    for (int k = 0; k < D - 1; ++k) load(k, k);
    for (int i = 0; i < steps; i += D) {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        load((k + D - 1) % D, i + k + D - 1);
        __builtin_amdgcn_sched_barrier(0);
        if (i + k < steps) step(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // merge the waves: maxima, then the scaled sums in wave order
  float* red = reinterpret_cast<float*>(lds);                       // [waves][16][128]
  float* ml = red + kAbsorbWaves * 16 * kAbsorbCols;                // [waves][16][2]
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (lane < 16) {
    ml[(w * 16 + lane) * 2] = m;
    ml[(w * 16 + lane) * 2 + 1] = l;
  }
  __syncthreads();
  float M = ml[lq * 2];
#pragma unroll
  for (int k = 1; k < kAbsorbWaves; ++k) M = fmaxf(M, ml[(k * 16 + lq) * 2]);
  const float f = w < nblk ? exp2f(m - M) : 0.0f;  // a wave without steps adds nothing
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float fr = __shfl(f, 4 * lg + r, 64);
    float* dst = red + ((size_t)w * 16 + 4 * lg + r) * kAbsorbCols + 8 * lq;
    *reinterpret_cast<float4*>(dst) = make_float4(acc[0][r] * fr, acc[1][r] * fr, acc[2][r] * fr, acc[3][r] * fr);
    *reinterpret_cast<float4*>(dst + 4) = make_float4(acc[4][r] * fr, acc[5][r] * fr, acc[6][r] * fr, acc[7][r] * fr);
  }
  __syncthreads();
  // this range's (max, sum) per head
  float Mh = -INFINITY, lh = 0.0f;
  if (tid < a.n_q) {
#pragma unroll
    for (int k = 0; k < kAbsorbWaves; ++k) Mh = fmaxf(Mh, ml[(k * 16 + tid) * 2]);
#pragma unroll
    for (int k = 0; k < kAbsorbWaves; ++k)
      lh += k < nblk ? ml[(k * 16 + tid) * 2 + 1] * exp2f(ml[(k * 16 + tid) * 2] - Mh) : 0.0f;
  }
  // a thread's 4 columns c.. of head h of the workgroup's sum; the slice's
  // finished sums go out times gamma as two bf16 parts
  const int HC = a.n_q * (kAbsorbCols / 4);
  auto sum4 = [&](int h, int c) {
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < kAbsorbWaves; ++k) {
      const float4 x = *reinterpret_cast<const float4*>(red + ((size_t)k * 16 + h) * kAbsorbCols + c);
      o.x += x.x, o.y += x.y, o.z += x.z, o.w += x.w;
      if constexpr (PACK) {
        const float4 y = *reinterpret_cast<const float4*>(red + ((size_t)k * 16 + h + 8) * kAbsorbCols + c);
        o.x += y.x, o.y += y.y, o.z += y.z, o.w += y.w;
      }
    }
    return o;
  };
  auto emit = [&](int h, int c, float4 o) {
    const int dc = sl * kAbsorbCols + c;
    if (dc >= a.d) return;
    if (a.fold == 0) {
      const uint2 gw = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.gamma) + dc);
      o.x *= bf_lo(gw.x), o.y *= bf_hi(gw.x), o.z *= bf_lo(gw.y), o.w *= bf_hi(gw.y);
    }
    uint2 hi, lo;
    hi.x = pack_bf16x2(o.x, o.y);
    hi.y = pack_bf16x2(o.z, o.w);
    lo.x = pack_bf16x2(o.x - bf_lo(hi.x), o.y - bf_hi(hi.x));
    lo.y = pack_bf16x2(o.z - bf_lo(hi.y), o.w - bf_hi(hi.y));
    uint16_t* dst = a.uh + ((size_t)b * a.n_q + h) * 2 * a.d + dc;
    *reinterpret_cast<uint2*>(dst) = hi;
    *reinterpret_cast<uint2*>(dst + a.d) = lo;
  };
  if (a.S == 1) {
    for (int e = tid; e < HC; e += NT) emit(e / (kAbsorbCols / 4), 4 * (e % (kAbsorbCols / 4)), sum4(e / (kAbsorbCols / 4), 4 * (e % (kAbsorbCols / 4))));
    if (sl == 0 && tid < a.n_q) {
      a.uml[((size_t)b * a.n_q + tid) * 2] = Mh;
      a.uml[((size_t)b * a.n_q + tid) * 2 + 1] = lh;
    }
    return;
  }
  // partials of (b, slice, range) meet in the workspace; the slice's last range
  // to arrive adds them in range order
  float* up = a.u + (((size_t)b * n_sl + sl) * a.S) * a.n_q * (kAbsorbCols + 2);
  const size_t rs = (size_t)a.n_q * (kAbsorbCols + 2);  // one range: sums [n_q][128], then (max, sum) [n_q][2]
  for (int e = tid; e < HC; e += NT) {
    const int h = e / (kAbsorbCols / 4), c = 4 * (e % (kAbsorbCols / 4));
    const float4 o = sum4(h, c);
    float* dst = up + s * rs + h * kAbsorbCols + c;
    store_dev(dst, o.x);
    store_dev(dst + 1, o.y);
    store_dev(dst + 2, o.z);
    store_dev(dst + 3, o.w);
  }
  if (tid < a.n_q) {
    store_dev(up + s * rs + a.n_q * kAbsorbCols + 2 * tid, Mh);
    store_dev(up + s * rs + a.n_q * kAbsorbCols + 2 * tid + 1, lh);
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this thread's partial is written
  __syncthreads();
  unsigned* ctr = a.done + (size_t)b * n_sl + sl;
  unsigned* bc = reinterpret_cast<unsigned*>(red);
  if (tid == 0) *bc = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (*bc != (unsigned)a.S - 1) return;
  float* ws = red + 4;  // [n_q][S] weights
  if (tid < a.n_q) {
    float mk[kAbsorbMaxRanges], lk[kAbsorbMaxRanges];
#pragma unroll
    for (int k = 0; k < kAbsorbMaxRanges; ++k) {
      const float* p = up + min(k, a.S - 1) * rs + a.n_q * kAbsorbCols + 2 * tid;
      mk[k] = load_dev(p);
      lk[k] = load_dev(p + 1);
    }
    float mm = mk[0], ll = 0.0f;
#pragma unroll
    for (int k = 1; k < kAbsorbMaxRanges; ++k) mm = fmaxf(mm, mk[k]);
#pragma unroll
    for (int k = 0; k < kAbsorbMaxRanges; ++k) {
      const float e = exp2f(mk[k] - mm);
      if (k < a.S) {
        ll = fmaf(lk[k], e, ll);
        ws[tid * kAbsorbMaxRanges + k] = e;
      }
    }
    if (sl == 0) {
      a.uml[((size_t)b * a.n_q + tid) * 2] = mm;
      a.uml[((size_t)b * a.n_q + tid) * 2 + 1] = ll;
    }
  }
  __syncthreads();
  for (int e = tid; e < HC; e += NT) {
    const int h = e / (kAbsorbCols / 4), c = 4 * (e % (kAbsorbCols / 4));
    float v[kAbsorbMaxRanges][4];
#pragma unroll
    for (int k = 0; k < kAbsorbMaxRanges; ++k)
      if (k < a.S) {
#pragma unroll
        for (int x = 0; x < 4; ++x) v[k][x] = load_dev(up + k * rs + h * kAbsorbCols + c + x);
      }
    float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < kAbsorbMaxRanges; ++k)
      if (k < a.S) {
        const float wt = ws[h * kAbsorbMaxRanges + k];
        o.x = fmaf(wt, v[k][0], o.x), o.y = fmaf(wt, v[k][1], o.y), o.z = fmaf(wt, v[k][2], o.z), o.w = fmaf(wt, v[k][3], o.w);
      }
    emit(h, c, o);
  }
}

// ------------------------------------------------------------------ value projection and merge

// One workgroup: 16 rows of W_v for up to 16 (sequence, query head) columns of
// the rows' KV head.  The 16 waves split d; each wave multiplies its 32-wide
// steps with both bf16 parts of the residual sums, every load in flight at
// once; the waves' sums meet in LDS in wave order, where the stored tail's
// partials join and the softmax denominator is applied.  Latency-bound: one
// round trip, 4.2 us at B = 1 (merging the ranges here instead, in every
// workgroup, took 16-18 us).
template <int HD, bool PACKED>
__global__ __launch_bounds__(64 * kVprojWaves, 1) void vproj_kernel(AbsorbArgs a, int seqs) {
  extern __shared__ __align__(16) float sm[];
  constexpr int NW = kVprojWaves;
  constexpr int NI = 5;  // steps per wave and pass: 80 steps of 32, d = 2560 in one pass
  float* red = sm;                    // [NW][16 cols][16 rows + 1]
  float* wts = sm + NW * 16 * 17;     // [16][P] weights of a column's P = 1 + n_tail states
  const int P = 1 + a.n_tail;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
  const int lq = lane & 15, lg = lane >> 4;
  const int g = a.n_q / a.n_kv;
  const int R0 = blockIdx.x * 16, j = R0 / HD;
  const int b0 = blockIdx.y * seqs;
  const int ncol = min(seqs, a.B - b0) * g;
  const int nst = a.d / 32;
  const uint16_t* wv = static_cast<const uint16_t*>(a.w_v);
  const uint16_t* wp = PACKED ? wv + ((size_t)(R0 >> 5) * (a.d / 16) + (lg >> 1)) * 512 +
                                    8 * ((R0 & 16) + lq + 32 * (lg & 1))
                              : wv + (size_t)(R0 + lq) * a.d + 8 * lg;
  const int cq = min(lq, ncol - 1);
  const uint16_t* ub = a.uh + ((size_t)(b0 + cq / g) * a.n_q + (size_t)j * g + cq % g) * 2 * a.d + 8 * lg;
  bf16x8_t A[NI], U[NI], V[NI];
  auto load = [&](int base) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int st = min(base + w + NW * i, nst - 1);
      A[i] = *reinterpret_cast<const bf16x8_t*>(wp + (size_t)st * (PACKED ? 1024 : 32));
      U[i] = *reinterpret_cast<const bf16x8_t*>(ub + 32 * st);
      V[i] = *reinterpret_cast<const bf16x8_t*>(ub + a.d + 32 * st);
    }
  };
  load(0);
  if (w < ncol) {  // wave c: the weights of column c
    const size_t row = (size_t)(b0 + w / g) * a.n_q + (size_t)j * g + w % g;
    float M = -INFINITY, den = 0.0f;
    for (int i = lane; i < P; i += 64) M = fmaxf(M, i < 1 ? a.uml[row * 2] : a.tml[(row * a.n_tail + i - 1) * 2]);
    M = wave_max(M);
    for (int i = lane; i < P; i += 64) {
      const float* s = i < 1 ? a.uml + row * 2 : a.tml + (row * a.n_tail + i - 1) * 2;
      const float e = exp2f(s[0] - M);
      den = fmaf(s[1], e, den);
      wts[w * P + i] = e;
    }
    den = wave_sum(den);
    for (int i = lane; i < P; i += 64) wts[w * P + i] /= den;
  }
  f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int base = 0; base < nst; base += NW * NI) {
    if (base > 0) load(base);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (base + w + NW * i < nst) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i], U[i], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i], V[i], acc, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[(w * 16 + lq) * 17 + 4 * lg + r] = acc[r];
  __syncthreads();
  const int c = tid >> 4, r = tid & 15;
  if (c >= ncol) return;
  const size_t row = (size_t)(b0 + c / g) * a.n_q + (size_t)j * g + c % g;
  const int f = R0 % HD + r;
  float o = 0.0f;
#pragma unroll
  for (int k = 0; k < NW; ++k) o += red[(k * 16 + c) * 17 + r];
  o *= wts[c * P];
#pragma unroll 8
  for (int t = 0; t < a.n_tail; ++t)
    o = fmaf(wts[c * P + 1 + t], a.tacc[(row * a.n_tail + t) * HD + f], o);
  static_cast<uint16_t*>(a.out)[row * HD + f] = from_f<uint16_t>(o);
}

// ------------------------------------------------------------------ launchers

template <class Tile, int HD, int RW, int MT, bool FOLD>
static hipError_t score_t(const AbsorbArgs& a, hipStream_t st) {
  if ((a.n_kv * HD) % RW != 0) return hipErrorInvalidValue;
  const size_t bytes = score_lds(HD, a.n_q / a.n_kv, RW, MT, a.d).end;
  static std::atomic<size_t> done{0};
  auto k = score_kernel<Tile, HD, RW, MT, FOLD>;
  hipError_t e = ensure_lds(k, bytes, done);
  if (e != hipSuccess) return e;
  const int n_rg = a.n_kv * HD / RW;
  const XcdMap m = xcd_map((long long)n_rg * a.B * ((a.T + MT - 1) / MT));
  int hg = 1;
  while (n_rg % (2 * hg) == 0 && (long long)(2 * hg) * (2 * hg) * RW <= (long long)MT * m.per) hg *= 2;
  hipLaunchKernelGGL(k, dim3(m.grid), dim3(Tile::NT), bytes, st, a, m.per, hg);
  return hipGetLastError();
}

template <int HD, int L>
static hipError_t score_l(const AbsorbArgs& a, int tile, hipStream_t st) {
  constexpr bool P = L != 0, F = L == 2;
  constexpr int LD = kv_ld<uint16_t>(256);
  switch (tile) {
    case kScore512x64: return score_t<WideTile<256, 64, P, F, 512, LD, false, true>, HD, 512, 64, F>(a, st);
    case kScore256x128: return score_t<WideTile<256, 128, P, F, 512, LD, true, false>, HD, 256, 128, F>(a, st);
    case kScore256x64: return score_t<WideTile<256, 64, P, F, 512, LD, true, false>, HD, 256, 64, F>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <int HD, bool PACK>
static hipError_t absorb_t(const AbsorbArgs& a, hipStream_t st) {
  const int rows = a.T_tail >= 64 ? 68 : (a.T_tail + 3) / 4 * 4;
  const int g = a.n_q / a.n_kv;
  const size_t main_b = sizeof(float) * (kAbsorbWaves * 16 * kAbsorbCols + kAbsorbWaves * 32);
  const size_t tail_b =
      a.n_tail > 0 ? attn_lds(align_up(sizeof(uint16_t) * (size_t)rows * kv_ld<uint16_t>(HD), 16), g, HD, rows).end : 0;
  const size_t bytes = main_b > tail_b ? main_b : tail_b;
  static std::atomic<size_t> done{0};
  auto k = absorb_kernel<HD, PACK>;
  hipError_t e = ensure_lds(k, bytes, done);
  if (e != hipSuccess) return e;
  const long long n = (long long)a.n_tail * a.n_kv * a.B +
                      (long long)((a.d + kAbsorbCols - 1) / kAbsorbCols) * a.S * a.B;
  hipLaunchKernelGGL(k, dim3((unsigned)n), dim3(64 * kAbsorbWaves), bytes, st, a, rows);
  return hipGetLastError();
}

template <int HD, int L>
static hipError_t vproj_t(const AbsorbArgs& a, hipStream_t st) {
  const int seqs = 16 / (a.n_q / a.n_kv);
  const size_t bytes = sizeof(float) * ((size_t)kVprojWaves * 16 * 17 + 16 * (size_t)(1 + a.n_tail));
  static std::atomic<size_t> done{0};
  auto k = vproj_kernel<HD, L != 0>;
  hipError_t e = ensure_lds(k, bytes, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(a.n_kv * HD / 16, (a.B + seqs - 1) / seqs), dim3(64 * kVprojWaves), bytes, st, a, seqs);
  return hipGetLastError();
}

template <int HD, int L>
static hipError_t absorb_l(const AbsorbArgs& a, int tile, hipStream_t st) {
  hipError_t e = score_l<HD, L>(a, tile, st);
  if (e == hipSuccess) e = a.n_q <= 8 ? absorb_t<HD, true>(a, st) : absorb_t<HD, false>(a, st);
  return e == hipSuccess ? vproj_t<HD, L>(a, st) : e;
}

hipError_t launch_absorb(const AbsorbArgs& a, int layout, int tile, hipStream_t st) {
  if (a.n_q > 16 || a.S < 1 || a.S > kAbsorbMaxRanges) return hipErrorInvalidValue;
  switch (layout) {
    case 0: return absorb_l<256, 0>(a, tile, st);
    case 1: return absorb_l<256, 1>(a, tile, st);
    case 2: return absorb_l<256, 2>(a, tile, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kvd
