// GEMMs over many token rows (prompts, verification of more than 16 rows, the shadow head over every layer's rows):
// bf16 weights times activations split into bf16 high + low parts, fp32 accumulation, with the epilogues fused.
#include "del_device.h"
#include <hip/hip_ext.h>

#include <algorithm>

namespace del {

namespace {

constexpr int WQ = 4;          // row blocks whose sums of squares go out as one number

// What a lane needs to know about its token row in an epilogue.
struct RowCtx {
  int row;          // token row of the pass
  bool valid;       // row < M
  int cb, token;    // block of 16 token rows, row inside it
  int pos;          // cache position (EPI_QKV)
  float sc;         // RMS scale
};

// RMS scale of token row `row` from the sums of squares its producer left (ssq_nb numbers per row, summed by the four
// lanes that share the row), or from p.rowscale.
__device__ __forceinline__ float row_scale(const GemmP& p, int row, int g) {
  if (p.ssq_in) {
    const float* s = p.ssq_in + (size_t)row * p.ssq_nb;
    float q = 0.f;
    for (int b = g; b < p.ssq_nb; b += 4) q += s[b];
    q += __shfl_xor(q, 16);
    q += __shfl_xor(q, 32);
    return 1.0f / sqrtf(q / (float)p.K + p.eps);
  }
  return p.rowscale ? p.rowscale[row] : 1.0f;
}

// Finished products of four consecutive row blocks nb0..nb0+3 for 16 token rows, straight from the matrix-core result
// layout: lane (g = lane / 16, token = lane % 16) holds rows 4g..4g+3 of every block for its token.  All of a lane's
// loads go out before its first store.
template <int EPI>
__device__ __forceinline__ void epilogue_quad(const GemmP& p, int nb0, const floatx4* acc, const RowCtx& r, int g) {
  float v[WQ][4];
#pragma unroll
  for (int i = 0; i < WQ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) v[i][j] = acc[i][j] * r.sc;
  const int row = r.valid ? r.row : 0;
  if (EPI == EPI_RESID) {
    float4 res[WQ], gain[WQ];
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
      const int n0 = min(nb0 + i, p.NB - 1) * 16 + 4 * g;     // rows of the residual are padded to whole blocks
      res[i] = *(const float4*)(p.R + (size_t)row * p.ldr + n0);
      if (p.XsOut) gain[i] = *(const float4*)(p.gain_out + n0);
    }
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
      const int n0 = (nb0 + i) * 16 + 4 * g;
      float o[4] = {v[i][0] + res[i].x, v[i][1] + res[i].y, v[i][2] + res[i].z, v[i][3] + res[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n0 + j >= p.N) o[j] = 0.f;     // padding
      if (r.valid && nb0 + i < p.NB) {
        *(float4*)(p.Y + (size_t)r.row * p.ldy + n0) = make_float4(o[0], o[1], o[2], o[3]);
        if (p.XsOut) {
          q += o[0] * o[0] + o[1] * o[1] + o[2] * o[2] + o[3] * o[3];
          const float w[4] = {o[0] * gain[i].x, o[1] * gain[i].y, o[2] * gain[i].z, o[3] * gain[i].w};
          uint2 hi, lo;
          split4(w, hi, lo);
          uint16_t* d = p.XsOut + (size_t)r.cb * p.xs_out_cb_stride + (size_t)(n0 >> 5) * 1024 +
                        (((n0 & 31) >> 3) * 16 + r.token) * 8 + (n0 & 7);
          *(uint2*)d = hi;
          *(uint2*)(d + 512) = lo;
        }
      }
    }
    if (p.ssq_out) {
      q += __shfl_xor(q, 16);
      q += __shfl_xor(q, 32);
      if (g == 0 && r.valid && nb0 < p.NB) p.ssq_out[(size_t)r.row * ((p.NB + WQ - 1) / WQ) + nb0 / WQ] = q;
    }
  } else if (EPI == EPI_QKV) {
    const int hd = p.hd, half = hd >> 1;
    float4 c0[WQ], c1[WQ];
#pragma unroll
    for (int i = 0; i < WQ; ++i) {   // (cos, sin) of this lane's four rotary pairs
      const int v0 = min(nb0 + i, p.NB - 1) * 16, s0 = v0 % hd;
      const float4* t = (const float4*)(p.rope + (size_t)r.pos * half + (s0 >> 4) * 8 + 4 * (g & 1));
      const bool rotary = v0 / hd < p.n_q + p.n_kv;           // uniform
      c0[i] = rotary ? t[0] : make_float4(0.f, 0.f, 0.f, 0.f);
      c1[i] = rotary ? t[1] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
      const int v0 = (nb0 + i) * 16, hh = v0 / hd, s0 = v0 - hh * hd;
      if (nb0 + i >= p.NB) continue;                          // uniform
      if (hh < p.n_q + p.n_kv) {
        // rows 0..7 of a block are features j, rows 8..15 their partners j + hd/2, held 32 lanes further on
        float o[4];
        const float cs[8] = {c0[i].x, c0[i].y, c0[i].z, c0[i].w, c1[i].x, c1[i].y, c1[i].z, c1[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float other = __shfl_xor(v[i][j], 32);
          o[j] = g < 2 ? v[i][j] * cs[2 * j] - other * cs[2 * j + 1] : v[i][j] * cs[2 * j] + other * cs[2 * j + 1];
        }
        const int f = (s0 >> 4) * 8 + 4 * (g & 1) + (g < 2 ? 0 : half);
        if (r.valid) {
          if (hh < p.n_q) {
            *(float4*)(p.Q + (size_t)r.row * p.ldq + hh * hd + f) = make_float4(o[0], o[1], o[2], o[3]);
          } else {
            uint16_t* k = (uint16_t*)p.Kc + ((size_t)(hh - p.n_q) * p.Tcap + r.pos) * hd + f;
            *(uint2*)k = make_uint2((uint32_t)f32_to_bf16_rne(o[0]) | ((uint32_t)f32_to_bf16_rne(o[1]) << 16),
                                    (uint32_t)f32_to_bf16_rne(o[2]) | ((uint32_t)f32_to_bf16_rne(o[3]) << 16));
          }
        }
      } else if (r.valid) {
        const int hv = hh - p.n_q - p.n_kv, f = s0 + 4 * g;
        uint16_t b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = f32_to_bf16_rne(v[i][j]);
        *(uint2*)((uint16_t*)p.Vc + ((size_t)hv * p.Tcap + r.pos) * hd + f) =
            make_uint2((uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16));
        if (p.VcT) {
          uint16_t* t = (uint16_t*)p.VcT + ((size_t)hv * hd + f) * p.TcapT + r.pos;
#pragma unroll
          for (int j = 0; j < 4; ++j) t[(size_t)j * p.TcapT] = b[j];
        }
      }
    }
  } else {   // EPI_SWIGLU: rows 0..7 of a block are gates, rows 8..15 the matching up projections
#pragma unroll
    for (int i = 0; i < WQ; ++i) {
      float a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float up = __shfl_xor(v[i][j], 32);
        a[j] = v[i][j] / (1.0f + expf(-v[i][j])) * up;
      }
      const int k8 = nb0 + i;                                 // eight activations per block
      if (g < 2 && r.valid && k8 < p.NB) {
        uint2 hi, lo;
        split4(a, hi, lo);
        uint16_t* d = p.XsOut + (size_t)r.cb * p.xs_out_cb_stride + (size_t)(k8 >> 2) * 1024 +
                      ((k8 & 3) * 16 + r.token) * 8 + 4 * g;
        *(uint2*)d = hi;
        *(uint2*)(d + 512) = lo;
      }
    }
  }
}

template <int EPI>
__device__ __forceinline__ RowCtx row_ctx(const GemmP& p, int cb, int lane) {
  RowCtx r;
  r.cb = cb;
  r.token = lane & 15;
  r.row = cb * 16 + r.token;
  r.valid = r.row < p.M;
  r.pos = 0;
  if (EPI == EPI_QKV) r.pos = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off + (r.valid ? r.row : 0);
  r.sc = 1.0f;
  return r;
}

// Best logit, its lowest index and the soft-max sum relative to it over the 16 * RW matrix rows a wave holds of one token
// row, as partial nb0 / RW of that row.  The positive RMS scale cannot change the arg-max; it is applied because the
// stored maximum and the sums are in logit units.
template <int RW, int CBW>
__device__ __forceinline__ void argmax_group(const GemmP& p, const floatx4 (&acc)[RW][CBW], int c, int nb0, int row, int g) {
  const float sc = row < p.M && p.rowscale ? p.rowscale[row] : 1.0f;
  float best = -INFINITY;
  int bi = 0x7FFFFFFF;
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = (nb0 + r) * 16 + 4 * g + j;
      const float v = acc[r][c][j] * sc;
      if (n < p.N && v > best) { best = v; bi = n; }   // ascending n: strict > keeps the lowest index
    }
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const float ov = __shfl_xor(best, o);
    const int oi = __shfl_xor(bi, o);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  float se = 0.f;
  if (p.psum) {
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((nb0 + r) * 16 + 4 * g + j < p.N) se += expf(acc[r][c][j] * sc - best);
    se += __shfl_xor(se, 16);
    se += __shfl_xor(se, 32);
  }
  if (g == 0 && row < p.M) {
    const size_t o = (size_t)row * ((p.NB + RW - 1) / RW) + nb0 / RW;
    p.pval[o] = best;
    p.pidx[o] = bi;
    if (p.psum) p.psum[o] = se;
  }
}

// Contiguous share of n units for the work-groups with index b % 8 == x (one XCD under round-robin dispatch); false: none.
__device__ __forceinline__ bool xcd_unit(int b, int n, int& u) {
  const int x = b & 7, lo = (int)((long long)n * x / 8), hi = (int)((long long)n * (x + 1) / 8);
  u = lo + (b >> 3);
  return u < hi;
}

}  // namespace

// One work-group of four waves = a tile of 2 RW row blocks of the matrix (256 or 128 rows) x CBT blocks of 16 token rows,
// wave (wr, wc) owning RW row blocks x CBT / 2 token blocks of it.  Weight and activation tiles are stored in operand order,
// so a k tile goes from memory straight into LDS (no registers) and every operand read is 1 KiB in lane order, free of
// bank conflicts.  What limits the main loop is LDS traffic against the matrix pipes: per k tile a work-group writes
// 2 RW + 2 CBT KiB and reads 4 x (RW + CBT) KiB for 4 RW x CBT instructions, 96 B per clock of matrix work at
// RW = CBT = 8, 144 at RW = 4 (measured ceiling of ds_read_b128: 119 B per clock).  Two to four stages, two
// work-groups per CU: while one waits at the barrier the other multiplies.
// Measured in us per launch against the form before it (8 row blocks x 128 or 256 token rows, one k tile of activations
// in registers, no splits): 7B shape at 1024 rows QKV 225 -> 176, gate/up 348 -> 298 (1.24 PFLOP/s of matrix
// instructions), output and down together 260 -> 244; 1B shape at 93 rows QKV 36 -> 16, gate/up 73 -> 28, output and
// down together 145 -> 35.  Loads alone take 0.74 of a launch's time and multiplication with its LDS reads 0.80: they overlap for
// the most part; a large product of the vendor library reaches 1.1 to 1.5 PFLOP/s on the same card.
// Tiles [0, plan.full) run over all k; the others are split into plan.S ranges of k, whose partial results
// wide_finish_k adds up in order.
template <int EPI, int RW, int CBT>
__global__ void __launch_bounds__(256, 2) gemm_wide_k(GemmP p, WidePlan w) {
  constexpr int WRB = 2 * RW;                        // row blocks per tile
  constexpr int CBW = CBT / 2;                       // token blocks per wave
  constexpr int WP = WRB / 4;                        // weight pieces (1 KiB) a wave stages per k tile
  constexpr int STAGE = WRB * 64 + CBT * 128;        // 16-byte pieces
  constexpr int AP = 2 * CBT / 4;                    // activation pieces (1 KiB) a wave stages per k tile
  // stages: as many as leave room for two work-groups per CU
  constexpr int NST = STAGE * 16 * 4 <= 81920 ? 4 : STAGE * 16 * 3 <= 81920 ? 3 : 2;
  // one array per stage: the compiler then knows that the loads filling one stage do not touch the one being read
  __shared__ __align__(16) uint4 st0[STAGE];
  __shared__ __align__(16) uint4 st1[STAGE];
  __shared__ __align__(16) uint4 st2[NST > 2 ? STAGE : 1];
  __shared__ __align__(16) uint4 st3[NST > 3 ? STAGE : 1];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4;
  const int wr = wave & 1, wc = wave >> 1;
  const int NB = p.NB, KT = p.KT, CB = (p.M + 15) >> 4;
  int b = blockIdx.x, tile, part = -1, k0 = 0, k1 = KT;
  const int gfull = (w.full + 7) / 8 * 8;
  if (b < gfull) {
    if (!xcd_unit(b, w.full, tile)) return;
  } else {
    if (!xcd_unit(b - gfull, w.rem * w.S, part)) return;
    const int s = part / w.rem;                      // neighbours share a k range
    tile = w.full + part - s * w.rem;
    k0 = (int)((long long)KT * s / w.S);
    k1 = (int)((long long)KT * (s + 1) / w.S);
    if (w.S == 1) part = -1;
  }
  const int slab = tile / w.NCG, cg = tile - slab * w.NCG;
  const int nb0 = slab * WRB, cb0 = cg * CBT;
  // sources are clamped (row blocks past the matrix, token blocks past the pass): their products are dropped
  typedef const void __attribute__((address_space(1)))* gptr_t;
  typedef void __attribute__((address_space(3)))* lptr_t;
  const uint4* Wt = (const uint4*)p.Wt;
  const uint4* Xs = (const uint4*)p.Xs;
  size_t wsrc[WP], xsrc[AP];
#pragma unroll
  for (int i = 0; i < WP; ++i) wsrc[i] = (size_t)min(nb0 + wave * WP + i, NB - 1) * KT * 64;
#pragma unroll
  for (int i = 0; i < AP; ++i) {
    const int q = wave * AP + i;
    xsrc[i] = (size_t)min(cb0 + (q >> 1), CB - 1) * KT * 128 + (q & 1) * 64;
  }
  auto request = [&](int kt, uint4* st) {
#pragma unroll
    for (int i = 0; i < WP; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(Wt + wsrc[i] + (size_t)kt * 64 + lane), (lptr_t)(st + (wave * WP + i) * 64), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < AP; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(Xs + xsrc[i] + (size_t)kt * 128 + lane),
                                       (lptr_t)(st + WRB * 64 + (wave * AP + i) * 64), 16, 0, 0);
  };
  floatx4 acc[RW][CBW];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int c = 0; c < CBW; ++c) acc[r][c] = (floatx4){0.f, 0.f, 0.f, 0.f};
  // the operands of token block c + 1 are read from LDS under block c's matrix instructions; the next stage's loads go
  // out once the first operands have been asked for
  auto multiply = [&](const uint4* st, auto&& request) {
    const uint4* ap = st + wr * RW * 64 + lane;
    const uint4* bp = st + WRB * 64 + wc * CBW * 128 + lane;
    uint4 a[RW], bh[2], bl[2];
    bh[0] = bp[0];
#pragma unroll
    for (int r = 0; r < RW; ++r) a[r] = ap[r * 64];
    bl[0] = bp[64];
    __builtin_amdgcn_sched_barrier(0);
    request();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      const int cur = c & 1, nxt = cur ^ 1;
      if (c + 1 < CBW) {
        bh[nxt] = bp[(c + 1) * 128];
        bl[nxt] = bp[(c + 1) * 128 + 64];
      }
#pragma unroll
      for (int r = 0; r < RW; ++r)
        acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[r]), __builtin_bit_cast(bf16x8, bh[cur]), acc[r][c], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < RW; ++r)
        acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[r]), __builtin_bit_cast(bf16x8, bl[cur]), acc[r][c], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);    // two LDS reads, then a block's matrix instructions
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * RW, 0);
    }
  };
  // one k tile: its stage has arrived for every wave once all have passed the barrier, which also says that the stage
  // of the tile before is no longer being read: it takes the tile NST - 1 further on.  Loads complete in order, so
  // leaving those of the NST - 2 younger stages in flight is enough.
  constexpr int LEFT = (NST - 2) * (WP + AP);
  static_assert(LEFT < 16, "the wait below sets the low four bits of vmcnt only");
  auto step = [&](int kt, const uint4* cur, uint4* nxt) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70 | LEFT);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    multiply(cur, [&]() { request(min(kt + NST - 1, k1 - 1), nxt); });   // (past the end: the last tile again, unused)
  };
  request(k0, st0);
  if (NST > 2) request(min(k0 + 1, k1 - 1), st1);
  if (NST > 3) request(min(k0 + 2, k1 - 1), st2);
  int kt = k0;
  if (NST == 2) {
    for (; kt + 2 <= k1; kt += 2) {
      step(kt, st0, st1);
      step(kt + 1, st1, st0);
    }
    if (kt < k1) step(kt, st0, st1);
  } else if (NST == 3) {
    for (; kt + 3 <= k1; kt += 3) {
      step(kt, st0, st2);
      step(kt + 1, st1, st0);
      step(kt + 2, st2, st1);
    }
    if (kt < k1) step(kt, st0, st2);
    if (kt + 1 < k1) step(kt + 1, st1, st0);
  } else {
    for (; kt + 4 <= k1; kt += 4) {
      step(kt, st0, st3);
      step(kt + 1, st1, st0);
      step(kt + 2, st2, st1);
      step(kt + 3, st3, st2);
    }
    if (kt < k1) step(kt, st0, st3);
    if (kt + 1 < k1) step(kt + 1, st1, st0);
    if (kt + 2 < k1) step(kt + 2, st2, st1);
  }
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);     // no load into LDS is left in flight
  if (part >= 0) {
    floatx4* o = (floatx4*)p.part + ((size_t)part * CBT + wc * CBW) * WRB * 64 + wr * RW * 64 + lane;
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int r = 0; r < RW; ++r) o[((size_t)c * WRB + r) * 64] = acc[r][c];
    return;
  }
  if (EPI == EPI_ARGMAX) {
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      const int cb = cb0 + wc * CBW + c;
      if (cb < CB && nb0 + wr * RW < NB) argmax_group<RW, CBW>(p, acc, c, nb0 + wr * RW, cb * 16 + (lane & 15), g);
    }
    return;
  }
#pragma unroll
  for (int c = 0; c < CBW; ++c) {
    const int cb = cb0 + wc * CBW + c;
    if (cb >= CB) break;
    RowCtx r = row_ctx<EPI>(p, cb, lane);
    if (EPI != EPI_RESID) r.sc = row_scale(p, r.valid ? r.row : 0, g);
#pragma unroll
    for (int q = 0; q < RW; q += WQ) {
      const floatx4 v[WQ] = {acc[q][c], acc[q + 1][c], acc[q + 2][c], acc[q + 3][c]};
      epilogue_quad<EPI>(p, nb0 + wr * RW + q, v, r, g);
    }
  }
}

// Adds the plan.S partial results of the split tiles, in order of k, and runs the epilogue: a wave = four row blocks x
// one block of 16 token rows.
template <int EPI>
__global__ void __launch_bounds__(256) wide_finish_k(GemmP p, WidePlan w) {
  const int WRB = 2 * w.RW, quads = WRB / WQ;
  const int lane = threadIdx.x & 63, g = lane >> 4, unit = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int quad = unit % quads, c = unit / quads % w.CBT, r0 = unit / quads / w.CBT;
  if (r0 >= w.rem) return;
  const int tile = w.full + r0, slab = tile / w.NCG, cb = (tile - slab * w.NCG) * w.CBT + c;
  const int nb0 = slab * WRB + quad * WQ;
  if (cb * 16 >= p.M || nb0 >= p.NB) return;
  const floatx4* src = (const floatx4*)p.part + (((size_t)r0 * w.CBT + c) * WRB + quad * WQ) * 64 + lane;
  const size_t stride = (size_t)w.rem * w.CBT * WRB * 64;
  RowCtx r = row_ctx<EPI>(p, cb, lane);
  if (EPI != EPI_RESID) r.sc = row_scale(p, r.valid ? r.row : 0, g);
  floatx4 v[WQ];
#pragma unroll
  for (int i = 0; i < WQ; ++i) v[i] = src[i * 64];
#pragma unroll 4
  for (int s = 1; s < w.S; ++s) {
#pragma unroll
    for (int i = 0; i < WQ; ++i) v[i] += src[s * stride + i * 64];
  }
  epilogue_quad<EPI>(p, nb0, v, r, g);
}

// How a launch is cut up: the cheapest plan of a small model of the kernel, whose constants are what it measured on
// matrices of 128 to 8016 row blocks and 64 to 896 k tiles with 8 to 1024 token rows (most plans within 15 %).  A k tile
// costs a work-group `alone` us when it has its CU to itself (a barrier and a memory latency per tile) and `shared` us
// per work-group when there are several (bound by what LDS and L2 deliver); the weights come in at HBM_BYTES_PER_US at
// best.  Splitting k adds a launch, a step per part and the partial results' way through the caches.  Per wave 8 row
// blocks read LDS least (large products); 4 give twice the tiles where those would not fill the chip.
// E.g. 256 row blocks, 344 k tiles (7B down projection): at 1024 rows 296 us unsplit, 171 in two, 161 in four ranges;
// at 256 rows 156 / 86 / 54 / 55 us with 1 / 2 / 4 / 8.  192 row blocks, 64 k tiles (1B QKV) at 256 rows: 20.0 us with 8
// row blocks per wave (two ranges), 13.8 with 4 (unsplit).
namespace {

struct Form { int RW, CBT; double alone, shared; int in_flight; };   // us per k tile; weight bytes on their way per work-group
constexpr Form forms[] = {{8, 2, 0.41, 0.36, 49152}, {8, 4, 0.55, 0.44, 32768}, {8, 8, 0.95, 0.76, 16384},
                          {4, 2, 0.18, 0.17, 24576}, {4, 4, 0.30, 0.27, 24576}, {4, 8, 0.56, 0.46, 16384}};

// The best number of k ranges for tiles of this form, NCG side by side; *us: its time.
WidePlan best_split(const Form& f, int NB, int KT, int NCG, int whole, double* us) {
  constexpr double START_US = 3.0, LAUNCH_US = 4.0, PER_PART_US = 0.25, HBM_BYTES_PER_US = 5.5e6, HBM_LATENCY_US = 0.8,
                   PART_BYTES_PER_US = 8.0e6;
  constexpr int CUS = 256, MAX_PART = 512, MAX_SPLIT = 32, MIN_KT = 4;
  WidePlan best{};
  *us = 1e30;
  const int wrb = 2 * f.RW, T = (NB + wrb - 1) / wrb * NCG;
  for (int S = 1; S <= MAX_SPLIT; ++S) {
    const int full = S > 1 ? T / CUS * CUS : T, rem = T - full;
    if (S > 1 && (whole || rem == 0 || S * MIN_KT > KT || rem * S > MAX_PART)) break;
    const int wgs = (full + CUS - 1) / CUS + (rem * S + CUS - 1) / CUS;   // work-groups of the busiest CU
    const double kts = (double)((full + CUS - 1) / CUS) * KT + (double)((rem * S + CUS - 1) / CUS) * ((KT + S - 1) / S);
    // the weights arrive as fast as the memory delivers, or as the requests that are out at one time allow
    const double resident = std::min(full + rem * S, 2 * CUS);
    const double rate = std::min(HBM_BYTES_PER_US, resident / NCG * f.in_flight / HBM_LATENCY_US);
    double t = std::max((wgs > 1 ? f.shared : f.alone) * kts, (double)NB * KT * 1024 / rate) + START_US;
    if (S > 1) t += LAUNCH_US + PER_PART_US * S + 2.0 * rem * S * f.CBT * wrb * 1024 / PART_BYTES_PER_US;
    if (t < *us) {
      *us = t;
      best = WidePlan{f.RW, f.CBT, NCG, full, rem, S};
    }
  }
  return best;
}

}  // namespace

WidePlan wide_plan(int NB, int KT, int M, int whole) {
  WidePlan best{};
  double best_t = 1e30;
  const int CB = (M + 15) / 16;
  for (const Form& f : forms) {
    double t;
    const WidePlan w = best_split(f, NB, KT, (CB + f.CBT - 1) / f.CBT, whole, &t);
    if (t < best_t) { best_t = t; best = w; }
  }
  return best;
}

// The most workspace that a plan for up to M token rows asks for.
size_t wide_part_most(int NB, int KT, int M, int whole) {
  size_t most = 0;
  const int CB = (M + 15) / 16;
  for (const Form& f : forms)
    for (int ncg = 1; ncg <= (CB + f.CBT - 1) / f.CBT; ++ncg) {
      double t;
      most = std::max(most, wide_part_bytes(best_split(f, NB, KT, ncg, whole, &t)));
    }
  return most;
}

size_t wide_part_bytes(const WidePlan& w) { return w.rem ? (size_t)w.rem * w.S * w.CBT * 2 * w.RW * 1024 : 0; }
int wide_ssq_nb(int NB) { return (NB + WQ - 1) / WQ; }

namespace {

template <int EPI, int RW, int CBT>
hipError_t launch_tile(const GemmP& p, const WidePlan& w, hipStream_t s) {
  const dim3 grid((w.full + 7) / 8 * 8 + (w.rem * w.S + 7) / 8 * 8), block(256);
  const bool split = w.rem > 0;
  hipExtLaunchKernelGGL((gemm_wide_k<EPI, RW, CBT>), grid, block, 0, s, p.ev_start, split ? nullptr : p.ev_stop, 0, p, w);
  if constexpr (EPI != EPI_ARGMAX)
    if (split)
      hipExtLaunchKernelGGL((wide_finish_k<EPI>), dim3((w.rem * w.CBT * (2 * RW / WQ) + 3) / 4), block, 0, s, nullptr,
                            p.ev_stop, 0, p, w);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_epi(const GemmP& p, const WidePlan& w, hipStream_t s) {
  if (w.RW == 8 && w.CBT == 8) return launch_tile<EPI, 8, 8>(p, w, s);
  if (w.RW == 8 && w.CBT == 4) return launch_tile<EPI, 8, 4>(p, w, s);
  if (w.RW == 8 && w.CBT == 2) return launch_tile<EPI, 8, 2>(p, w, s);
  if (w.RW == 4 && w.CBT == 8) return launch_tile<EPI, 4, 8>(p, w, s);
  if (w.RW == 4 && w.CBT == 4) return launch_tile<EPI, 4, 4>(p, w, s);
  if (w.RW == 4 && w.CBT == 2) return launch_tile<EPI, 4, 2>(p, w, s);
  return hipErrorInvalidValue;
}

}  // namespace

// Shadow-head GEMM with fused arg-max over p.M rows: p.pval / pidx / psum receive *n_parts partials per row.
hipError_t launch_gemm_wide_argmax(const GemmP& p, int* n_parts, hipStream_t s) {
  if (p.NB <= 0 || p.KT <= 0 || p.M < 1 || !p.pval || !p.pidx) return hipErrorInvalidValue;
  const WidePlan w = wide_plan(p.NB, p.KT, p.M, 1);
  *n_parts = (p.NB + w.RW - 1) / w.RW;
  return launch_gemm_wide(p, EPI_ARGMAX, w, s);
}

hipError_t launch_gemm_wide(const GemmP& p, int epi, hipStream_t s) {
  if (p.NB <= 0 || p.KT <= 0 || p.M < 1) return hipErrorInvalidValue;
  return launch_gemm_wide(p, epi, wide_plan(p.NB, p.KT, p.M, p.wide_form == 1), s);
}

hipError_t launch_gemm_wide(const GemmP& p, int epi, const WidePlan& w, hipStream_t s) {
  if (p.NB <= 0 || p.KT <= 0 || p.M < 1 || p.wdtype != 1 || !p.Xs) return hipErrorInvalidValue;
  if (w.rem > 0 && (!p.part || wide_part_bytes(w) > p.part_bytes)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_RESID: return launch_epi<EPI_RESID>(p, w, s);
    case EPI_QKV: return launch_epi<EPI_QKV>(p, w, s);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(p, w, s);
    case EPI_ARGMAX: return w.rem ? hipErrorInvalidValue : launch_epi<EPI_ARGMAX>(p, w, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace del
