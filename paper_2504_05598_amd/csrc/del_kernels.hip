// gfx950 (CDNA4) kernels of the greedy self-speculative decode round.
//
// Everything here is bound by HBM traffic except the multi-row GEMMs, which use the matrix
// cores.  Weights are streamed exactly once per launch in 1 KiB wave-sized tiles (see
// del_kernels.h); activations stay fp32 on the vector path and are split into bf16 hi + lo
// halves (16 mantissa bits together) on the matrix-core path, accumulating in fp32.
#include "del_device.h"
#include <hip/hip_ext.h>

namespace del {

constexpr int MAXW = 16;  // waves per work-group at most
constexpr int QBMAX = 32;  // query rows per attention batch at most

template <int KPL> struct WDec;
template <> struct WDec<8> {  // 8 bf16 in a uint4
  static __device__ __forceinline__ void dec(const uint4& w, float* f) {
    f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xFFFF0000u);
    f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xFFFF0000u);
    f[4] = __uint_as_float(w.z << 16); f[5] = __uint_as_float(w.z & 0xFFFF0000u);
    f[6] = __uint_as_float(w.w << 16); f[7] = __uint_as_float(w.w & 0xFFFF0000u);
  }
};
template <> struct WDec<4> {  // 4 fp32 in a uint4
  static __device__ __forceinline__ void dec(const uint4& w, float* f) {
    f[0] = __uint_as_float(w.x); f[1] = __uint_as_float(w.y);
    f[2] = __uint_as_float(w.z); f[3] = __uint_as_float(w.w);
  }
};

// One embedding row out of the tiled table as fp32: a row's k tile is four 16-byte pieces (lanes g*16 + r
// of the tile), so every thread moves whole pieces.  kpl = 8 (bf16) or 4 (fp32) elements per piece.
__device__ __forceinline__ void gather_embedding(const void* Et, int kpl, int KT, int id, float* out, int d_model,
                                                 int tid, int nthr) {
  const int nb = id >> 4, r = id & 15;
  const int pieces = (d_model + kpl - 1) / kpl;
  for (int c = tid; c < pieces; c += nthr) {
    const int kt = c >> 2, g = c & 3;
    const uint4 raw = ((const uint4*)Et)[((size_t)nb * KT + kt) * 64 + g * 16 + r];
    float v[8];
    if (kpl == 8) {
      WDec<8>::dec(raw, v);
    } else {
      v[0] = __uint_as_float(raw.x); v[1] = __uint_as_float(raw.y);
      v[2] = __uint_as_float(raw.z); v[3] = __uint_as_float(raw.w);
    }
    const int k0 = c * kpl;
    if (k0 + kpl <= d_model) {
      *(float4*)(out + k0) = make_float4(v[0], v[1], v[2], v[3]);
      if (kpl == 8) *(float4*)(out + k0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else {
      for (int e = 0; e < kpl && k0 + e < d_model; ++e) out[k0 + e] = v[e];
    }
  }
}

template <bool BF16> __device__ __forceinline__ void kv_store(void* base, size_t idx, float v) {
  if (BF16) ((uint16_t*)base)[idx] = f32_to_bf16_rne(v);
  else ((float*)base)[idx] = v;
}

// Eight consecutive features (a quarter of a 32-wide k tile) of one token row -> hi/lo split tiles.
// k8 = index of the group of eight (feature / 8).
__device__ __forceinline__ void split_store8(uint16_t* Xs, int k8, int token, const float* v) {
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const uint16_t h0 = f32_to_bf16_rne(v[e]), h1 = f32_to_bf16_rne(v[e + 1]);
    const uint16_t l0 = f32_to_bf16_rne(v[e] - bf16_bits_to_f32(h0));
    const uint16_t l1 = f32_to_bf16_rne(v[e + 1] - bf16_bits_to_f32(h1));
    hi[e >> 1] = (uint32_t)h0 | ((uint32_t)h1 << 16);
    lo[e >> 1] = (uint32_t)l0 | ((uint32_t)l1 << 16);
  }
  uint16_t* d = Xs + (size_t)(k8 >> 2) * 1024 + ((k8 & 3) * 16 + token) * 8;
  *(uint4*)d = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  *(uint4*)(d + 512) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

// ---------------------------------------------------------------------------------------
// Epilogues.  fin[mi][r] holds the finished 16 outputs of row-block nb for token row mi.
// ---------------------------------------------------------------------------------------
// WAVE: run by one wave on its own tile (thread index = lane) instead of the whole work-group.
// XsOut / ssq_out: where this block of 16 token rows puts its split tiles / sums of squares
// (token row mi of the block is row mi there).
template <int EPI, bool BF16KV, bool WAVE = false>
__device__ __forceinline__ void epilogue(const GemmP& p, int nb, float (*fin)[16], int m, int rowbase,
                                         uint16_t* XsOut, float* ssq_out) {
  const int nthr = WAVE ? 64 : blockDim.x;
  const int t0 = WAVE ? (threadIdx.x & 63) : threadIdx.x;
  if (EPI == EPI_STORE || EPI == EPI_RESID) {
    for (int tid = t0; tid < m * 16; tid += nthr) {
      const int mi = tid >> 4, r = tid & 15, n = nb * 16 + r;
      if (n < p.N) {
        float v = fin[mi][r];
        if (EPI == EPI_RESID) v += p.R[(size_t)(rowbase + mi) * p.ldr + n];
        p.Y[(size_t)(rowbase + mi) * p.ldy + n] = v;
        if (EPI == EPI_RESID && XsOut) fin[mi][r] = v;   // keep the residual-added value for the split below
      } else if (EPI == EPI_RESID && XsOut) {
        fin[mi][r] = 0.f;
      }
    }
    if (EPI == EPI_RESID && XsOut) {   // rowbase == 0 on this path (one block of <= 16 token rows)
      if (WAVE) __builtin_amdgcn_wave_barrier(); else __syncthreads();
      for (int tid = t0; tid < m * 2; tid += nthr) {
        const int mi = tid >> 1, half = tid & 1;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int n = nb * 16 + half * 8 + e;
          v[e] = fin[mi][half * 8 + e] * (p.gain_out ? p.gain_out[n] : 1.f);
        }
        split_store8(XsOut, nb * 2 + half, mi, v);
      }
      if (ssq_out) {
        for (int tid = t0; tid < m; tid += nthr) {
          float q = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) q += fin[tid][r] * fin[tid][r];
          ssq_out[(size_t)tid * p.NB + nb] = q;
        }
      }
    }
  } else if (EPI == EPI_QKV) {
    for (int tid = t0; tid < m * 16; tid += nthr) {
      const int mi = tid >> 4, r = tid & 15;
      const int hd = p.hd, half = hd >> 1;
      const int v0 = nb * 16;
      const int hh = v0 / hd, s0 = v0 - hh * hd;
      const int pos = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off + rowbase + mi;
      if (hh < p.n_q + p.n_kv) {  // rotary heads: rows r and r+8 are the pair (j, j + hd/2)
        if (r < 8) {
          const int j = (s0 >> 4) * 8 + r;
          const float a = fin[mi][r], b = fin[mi][r + 8];
          const float2 cs = p.rope[(size_t)pos * half + j];
          const float ar = a * cs.x - b * cs.y;
          const float br = b * cs.x + a * cs.y;
          if (hh < p.n_q) {
            float* q = p.Q + (size_t)(rowbase + mi) * p.ldq + hh * hd;
            q[j] = ar;
            q[j + half] = br;
          } else {
            const size_t base = ((size_t)(hh - p.n_q) * p.Tcap + pos) * hd;
            kv_store<BF16KV>(p.Kc, base + j, ar);
            kv_store<BF16KV>(p.Kc, base + j + half, br);
          }
        }
      } else {
        const size_t base = ((size_t)(hh - p.n_q - p.n_kv) * p.Tcap + pos) * hd;
        kv_store<BF16KV>(p.Vc, base + s0 + r, fin[mi][r]);
        if (BF16KV && p.VcT)
          ((uint16_t*)p.VcT)[((size_t)(hh - p.n_q - p.n_kv) * hd + s0 + r) * p.TcapT + pos] = f32_to_bf16_rne(fin[mi][r]);
      }
    }
  } else if (EPI == EPI_SWIGLU) {
    for (int tid = t0; tid < m * 8; tid += nthr) {
      const int mi = tid >> 3, r = tid & 7, j = nb * 8 + r;
      float a = 0.f;
      if (j < p.d_ffn) {
        const float gt = fin[mi][r], up = fin[mi][r + 8];
        a = gt / (1.0f + expf(-gt)) * up;
        p.ACT[(size_t)(rowbase + mi) * p.ldact + j] = a;
      }
      if (XsOut) {   // gather the 8 activations of this token row in one lane, store them split
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __shfl(a, (threadIdx.x & 56) + e);
        if (r == 0) split_store8(XsOut, nb, mi, v);
      }
    }
  } else if (EPI == EPI_ARGMAX) {
    for (int tid = t0; tid < m; tid += nthr) {
      const int mi = tid;
      float best = -INFINITY;
      int bi = 0x7FFFFFFF;
      for (int r = 0; r < 16; ++r) {
        const int n = nb * 16 + r;
        const float v = fin[mi][r];
        if (n < p.N && v > best) { best = v; bi = n; }  // strict >: lowest index wins ties
      }
      const size_t o = (size_t)(p.prow0 + rowbase + mi) * p.NB + nb;
      p.pval[o] = best;
      p.pidx[o] = bi;
      if (p.psum) {   // soft-max denominator of this block relative to its own maximum
        float se = 0.f;
        for (int r = 0; r < 16; ++r)
          if (nb * 16 + r < p.N) se += expf(fin[mi][r] - best);
        p.psum[o] = se;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Weight streaming.  A weight tile is read exactly once per launch, so it is fetched with a
// non-temporal load (no reuse: keeps the stream out of the way of the cached activations),
// and every wave owns a contiguous span of the k tiles of its row block.
// ---------------------------------------------------------------------------------------
constexpr int GU = 4;  // tiles in flight per wave and pipeline stage (x2: current + next)

// The k tiles of a row block are split over the waves in whole groups of `grp` tiles, as evenly as the
// group count allows; only the last wave can be left with fewer than `grp` tiles at its end.  (A
// remainder is loaded tile by tile with its latency exposed, so a split in tiles, which leaves one in
// every wave, costs about two memory latencies per launch.)
__device__ __forceinline__ void wave_span(int KT, int nw, int wave, int grp, int& lo, int& hi) {
  const int G = KT / grp;
  lo = (G * wave / nw) * grp;
  hi = wave == nw - 1 ? KT : (G * (wave + 1) / nw) * grp;
}

// ---------------------------------------------------------------------------------------
// The input row of the one-row output projection is the attention output, handed over as att_S <= ATT_SMAX
// per-split softmax partials (max, sum, weighted values): merged while the row is staged.  Request and merge
// are separate steps: all loads of a lane's four features go out at once, with the split index clamped
// instead of a branch around the load, so that a caller can put its weight-tile requests between the two and
// wait for the partials alone; the sums run over the splits in ascending order.
// ---------------------------------------------------------------------------------------
constexpr int ATT_SMAX = 8;
struct AttReq {
  float pm[ATT_SMAX], pl[ATT_SMAX];
  float4 pa[ATT_SMAX];
};
__device__ __forceinline__ void att_request(const GemmP& p, int k, AttReq& r) {
  const int kc = min(k, p.K - 4);            // features past K (padding) merge to zero: any valid address will do
  const int h = kc / p.att_hd, d = kc - h * p.att_hd;
  const size_t row = (size_t)h * p.att_stride;
#pragma unroll
  for (int s = 0; s < ATT_SMAX; ++s) {
    const int sc = min(s, p.att_S - 1);
    r.pm[s] = p.att_PM[row + sc];
    r.pl[s] = p.att_PL[row + sc];
    r.pa[s] = *(const float4*)(p.att_PA + (row + sc) * p.att_hd + d);
  }
}
__device__ __forceinline__ float4 att_merge(const GemmP& p, int k, const AttReq& r) {
  float mx = -INFINITY;
#pragma unroll
  for (int s = 0; s < ATT_SMAX; ++s)
    if (s < p.att_S) mx = fmaxf(mx, r.pm[s]);
  float L = 0.f;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int s = 0; s < ATT_SMAX; ++s)
    if (s < p.att_S) {
      const float ms = r.pm[s];
      const float c = ms > -INFINITY ? expf(ms - mx) : 0.f;
      L += c * r.pl[s];
      a.x += c * r.pa[s].x; a.y += c * r.pa[s].y; a.z += c * r.pa[s].z; a.w += c * r.pa[s].w;
    }
  const float inv = 1.0f / L;
  return k < p.K ? make_float4(a.x * inv, a.y * inv, a.z * inv, a.w * inv) : make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---------------------------------------------------------------------------------------
// Vector-ALU GEMV (M = 1) / skinny GEMM (M = 2; 4 and 8 with 32-bit weights): one work-group per 16-row block; each
// lane accumulates one weight row over its wave's span of k tiles, fp32 throughout.
// M = 1 (the draft path): the gained input row is staged once in LDS (dynamic, KT*TK floats)
// while the first weight tiles are already in flight; M > 1 reads the rows through the cache.
// ---------------------------------------------------------------------------------------
// One weight tile (16 rows x TK inputs, this lane's KPL elements) times the M input rows.
template <int KPL, int M>
__device__ __forceinline__ void valu_tile(const uint4& w, int kt, int g, const float* xs, const GemmP& p, bool has_gain,
                                          float* acc, float* ss) {
  constexpr int TK = 4 * KPL;
  float wf[KPL];
  WDec<KPL>::dec(w, wf);
  const int k0 = kt * TK + g * KPL;
  if (M == 1) {
#pragma unroll
    for (int e = 0; e < KPL; e += 4) {
      const float4 t = *(const float4*)(xs + k0 + e);
      acc[0] += wf[e] * t.x;
      acc[0] += wf[e + 1] * t.y;
      acc[0] += wf[e + 2] * t.z;
      acc[0] += wf[e + 3] * t.w;
    }
  } else {
    float gn[KPL];
#pragma unroll
    for (int e = 0; e < KPL; e += 4) {
      float4 t = has_gain ? *(const float4*)(p.gain + k0 + e) : make_float4(1.f, 1.f, 1.f, 1.f);
      gn[e] = t.x; gn[e + 1] = t.y; gn[e + 2] = t.z; gn[e + 3] = t.w;
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const float* xr = p.X + (size_t)m * p.ldx + k0;
#pragma unroll
      for (int e = 0; e < KPL; e += 4) {
        const float4 t = *(const float4*)(xr + e);
        ss[m] += t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w;
        acc[m] += wf[e] * (t.x * gn[e]);
        acc[m] += wf[e + 1] * (t.y * gn[e + 1]);
        acc[m] += wf[e + 2] * (t.z * gn[e + 2]);
        acc[m] += wf[e + 3] * (t.w * gn[e + 3]);
      }
    }
  }
}

// Waves per work-group by the number of input rows: every row adds an accumulator, a sum of squares and its
// share of the input row to a lane's registers, so the several-row forms run with fewer, larger-register waves
// (at 16 waves they spilled hundreds of registers).
template <int M> struct ValuWaves { static constexpr int max = M == 1 ? 16 : 4; };

// ATT: the input row is the attention output, still in per-split partials (the output projection of one row).  A form of
// its own: with both kinds of input row in one kernel a register was spilled, and the wait before its store (for the
// residual, ahead of the tile requests) cost every launch 1.1 us (7B down projection 19.1 us instead of 17.8).
template <int KPL, int M, int EPI, bool ATT = false>
__global__ void __launch_bounds__(64 * ValuWaves<M>::max) gemm_valu_k(GemmP p) {
  static_assert(!ATT || (M == 1 && EPI == EPI_RESID), "");
  constexpr int TK = 4 * KPL;
  extern __shared__ __align__(16) float xs[];
  __shared__ float red[MAXW][M][16];
  __shared__ float ssr[MAXW][M];
  __shared__ float fin[16][16];
  const int tid = threadIdx.x, nw = blockDim.x >> 6, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4;
  const int nb = blockIdx.x;
  float acc[M], ss[M];
#pragma unroll
  for (int m = 0; m < M; ++m) { acc[m] = 0.f; ss[m] = 0.f; }
  const bool has_gain = p.gain != nullptr;
  // this wave's span of k tiles: full groups of GU tiles (the last wave: plus a remainder of fewer than GU)
  int kt_lo, kt_hi;
  wave_span(p.KT, nw, wave, GU, kt_lo, kt_hi);
  const int ngroups = (kt_hi - kt_lo) / GU;
  const uint4* wp = (const uint4*)p.Wt + ((size_t)nb * p.KT + kt_lo) * 64 + lane;
  // Order of the first memory requests: the input row (it comes from the cache and is needed by every
  // wave before the first product), then two groups of GU weight tiles per wave (A: even groups, B: odd
  // groups).  Loads complete in order, so the row is in LDS and the barrier passed while the tiles are
  // still arriving, and every wave refills as soon as its own tiles are there; requested after the tiles,
  // the row would arrive behind the whole first burst of the grid and the memory pipe would run dry
  // while the work-group waits at the barrier.
  const int Kp = p.KT * TK, stride = blockDim.x * 4;
  float4 xv[4], gv[4];
  auto stage_load = [&](int base) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = base + j * stride;
      xv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      gv[j] = make_float4(1.f, 1.f, 1.f, 1.f);
      if (k < Kp) {
        xv[j] = *(const float4*)(p.X + k);
        if (has_gain) gv[j] = *(const float4*)(p.gain + k);
      }
    }
  };
  auto stage_store = [&](int base) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = base + j * stride;
      if (k < Kp) {
        const float4 x = xv[j], gg = gv[j];
        ss[0] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
        *(float4*)(xs + k) = make_float4(x.x * gg.x, x.y * gg.y, x.z * gg.z, x.w * gg.w);
      }
    }
  };
  // attention partials: those of a thread's first four features are asked for here, all at once, and merged when the tile
  // requests are out (merged split by split in a loop ahead of them, each split cost a memory round trip)
  AttReq rq;
  if constexpr (ATT) att_request(p, tid * 4, rq);
  else if (M == 1) stage_load(tid * 4);
  // one row: the residual, too, is requested up front (asked for in the epilogue it adds a memory round trip to every
  // launch: 0.8 us of the 5.3 a small matrix takes)
  float res = 0.f;
  if (M == 1 && EPI == EPI_RESID && tid < 16 && nb * 16 + tid < p.N) res = p.R[nb * 16 + tid];
  uint4 ta[GU], tb[GU];
  if (ngroups > 0) {
#pragma unroll
    for (int u = 0; u < GU; ++u) ta[u] = ld_stream(wp + u * 64);
  }
  if (ngroups > 1) {
#pragma unroll
    for (int u = 0; u < GU; ++u) tb[u] = ld_stream(wp + (GU + u) * 64);
  }
  if (M == 1) {
    // four 16-byte pieces per thread and batch: one batch covers 16 floats x threads, i.e. the whole row
    // for every shape but the widest rows on the smaller work-groups
    if constexpr (ATT) {
      for (int k = tid * 4; k < Kp; k += stride) {
        if (k != tid * 4) att_request(p, k, rq);
        const float4 x = att_merge(p, k, rq);
        ss[0] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
        *(float4*)(xs + k) = x;
      }
    } else {
      stage_store(tid * 4);
      for (int base = tid * 4 + 4 * stride; base < Kp; base += 4 * stride) {
        stage_load(base);
        stage_store(base);
      }
    }
    __syncthreads();
  }
  // Steady state: branch-free, and no register that a load is still filling is ever copied (a copy would
  // make the wave wait for every load in flight): group gi is used from A, A is refilled with group gi + 2,
  // then the same for B with gi + 1 and gi + 3, so two groups (2 * GU KiB per wave) stay in flight.
  auto use = [&](const uint4* tl, int gi) {
#pragma unroll
    for (int u = 0; u < GU; ++u) valu_tile<KPL, M>(tl[u], kt_lo + gi * GU + u, g, xs, p, has_gain, acc, ss);
  };
  auto fill = [&](uint4* tl, int gi) {
    const uint4* wn = wp + (size_t)gi * GU * 64;
#pragma unroll
    for (int u = 0; u < GU; ++u) tl[u] = ld_stream(wn + u * 64);
  };
  int gi = 0;
  for (; gi + 4 <= ngroups; gi += 2) {
    use(ta, gi);
    fill(ta, gi + 2);
    use(tb, gi + 1);
    fill(tb, gi + 3);
  }
  // one to three groups are left, the first two of them already requested
  const int left = ngroups - gi;
  if (left == 3) {
    use(ta, gi);
    fill(ta, gi + 2);
    use(tb, gi + 1);
    use(ta, gi + 2);
  } else if (left == 2) {
    use(ta, gi);
    use(tb, gi + 1);
  } else if (left == 1) {
    use(ta, gi);
  }
  for (int kt = kt_lo + ngroups * GU; kt < kt_hi; ++kt) {
    const uint4 w = ld_stream(wp + (size_t)(kt - kt_lo) * 64);
    valu_tile<KPL, M>(w, kt, g, xs, p, has_gain, acc, ss);
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    acc[m] += __shfl_xor(acc[m], 16);
    acc[m] += __shfl_xor(acc[m], 32);
    if (M == 1) {  // every thread staged a distinct slice: reduce over the whole wave
      for (int o = 1; o < 64; o <<= 1) ss[m] += __shfl_xor(ss[m], o);
    } else {       // lanes of one 16-lane group read the same k range: reduce over the groups
      ss[m] += __shfl_xor(ss[m], 16);
      ss[m] += __shfl_xor(ss[m], 32);
    }
  }
  if (lane < 16) {
#pragma unroll
    for (int m = 0; m < M; ++m) red[wave][m][lane] = acc[m];
  }
  if (lane == 0) {
#pragma unroll
    for (int m = 0; m < M; ++m) ssr[wave][m] = ss[m];
  }
  __syncthreads();
  for (int t = tid; t < M * 16; t += blockDim.x) {
    const int mi = t >> 4, r = t & 15;
    float s = 0.f;
    for (int w = 0; w < nw; ++w) s += red[w][mi][r];
    if (p.rms) {
      float q = 0.f;
      for (int w = 0; w < nw; ++w) q += ssr[w][mi];
      s *= 1.0f / sqrtf(q / (float)p.K + p.eps);
    }
    fin[mi][r] = M == 1 && EPI == EPI_RESID ? s + res : s;
  }
  __syncthreads();
  // (a row's residual is added by now; its split tiles are for the matrix-core path only)
  epilogue<M == 1 && EPI == EPI_RESID ? EPI_STORE : EPI, KPL == 8>(p, nb, fin, M, 0, p.XsOut, p.ssq_out);
}

// ---------------------------------------------------------------------------------------
// One-row GEMV, several row blocks per work-group (bf16 weights, KT = 16 * NG * GUX k tiles: 64 * NG with groups
// of 4 tiles, 160 with NG = 2 groups of 5): the grid is one
// work-group of 16 waves per compute unit and work-group w takes the row blocks w, w + grid, ...  The input
// row is staged once per work-group instead of once per row block, and a wave's tile requests run on across
// the row blocks: each wave owns NG groups of 4 tiles of every row block and keeps two groups in flight in two
// named register sets; the set just used is refilled at once, with the row block's later groups or the next
// row block's first ones, so the reduction and epilogue of a row block run under the next block's loads.  The
// loop over row blocks has no request behind a condition (the last block is a call of its own without refills),
// which lets the compiler keep exact wait counts (a wave waits for one tile at a time).  Against one row block
// per work-group: 17.9 -> 16.8 us (QKV), 30.2 -> 28.3 us (gate/up), 41.0 -> 39.1 us (head) in the measurement
// form of both kernels.
// ---------------------------------------------------------------------------------------
constexpr int ROWS_WAVES = 16;

template <int NG, int EPI, int GUX = GU>
__global__ void __launch_bounds__(1024) gemv_rows_k(GemmP p) {
  static_assert(NG >= 2 && NG % 2 == 0, "the two register sets take the groups of a row block in turn");
  constexpr int KPL = 8, TK = 32;
  extern __shared__ __align__(16) float xs[];
  __shared__ float red[2][ROWS_WAVES][16];
  __shared__ float ssr[ROWS_WAVES];
  __shared__ float fin[16][16];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4;
  const int wg = blockIdx.x, nwg = gridDim.x;
  if (wg >= p.NB) return;                                // uniform, before any barrier
  const int nblk = (p.NB - wg + nwg - 1) / nwg;          // row blocks of this work-group (>= 1)
  const int KT = p.KT;                                   // = 16 * NG * GUX (groups of GUX tiles: 4, or 5 for 160 k tiles)
  const int lo_t = wave * NG * GUX;                      // this wave's k tiles of every row block: [lo_t, lo_t + NG * GUX)
  const bool has_gain = p.gain != nullptr;
  float ss = 0.f;
  // the input row first (it comes from the cache and every wave needs it before its first product), then tiles.
  // The row has KP = KT * 32 floats: NJ float4 per thread, the last one only for the threads that still fall
  // inside the row.  Where it is the attention output, the partials of the first float4 are requested here and
  // merged once the tile requests are out.
  constexpr int XSTRIDE = 64 * ROWS_WAVES * 4, KP = ROWS_WAVES * NG * GUX * TK, NJ = (KP + XSTRIDE - 1) / XSTRIDE;
  auto inside = [&](int j) { return (j + 1) * XSTRIDE <= KP || tid * 4 + j * XSTRIDE < KP; };
  const bool att = p.att_S > 0;
  float4 xv[NJ], gv[NJ];
  AttReq rq;
  if (att) {
    att_request(p, tid * 4, rq);
  } else {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      // (a thread past the row's end reads the row's last float4 and drops it: no branch around the load)
      xv[j] = *(const float4*)(p.X + min(tid * 4 + j * XSTRIDE, KP - 4));
      if (!inside(j)) xv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    gv[j] = has_gain ? *(const float4*)(p.gain + min(tid * 4 + j * XSTRIDE, KP - 4)) : make_float4(1.f, 1.f, 1.f, 1.f);
  const size_t blk_stride = (size_t)nwg * KT * 64;
  const uint4* wp = (const uint4*)p.Wt + ((size_t)wg * KT + lo_t) * 64 + lane;   // this wave's first tile of the current row block
  uint4 ta[GUX], tb[GUX];
  auto fill = [&](uint4* t, const uint4* src) {
#pragma unroll
    for (int u = 0; u < GUX; ++u) t[u] = ld_stream(src + u * 64);
  };
  fill(ta, wp);
  fill(tb, wp + GUX * 64);
  if (att) {
    xv[0] = att_merge(p, tid * 4, rq);
#pragma unroll
    for (int j = 1; j < NJ; ++j) {
      xv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (inside(j)) {
        att_request(p, tid * 4 + j * XSTRIDE, rq);
        xv[j] = att_merge(p, tid * 4 + j * XSTRIDE, rq);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const float4 x = xv[j], gg = gv[j];
    ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
    if (inside(j)) *(float4*)(xs + tid * 4 + j * XSTRIDE) = make_float4(x.x * gg.x, x.y * gg.y, x.z * gg.z, x.w * gg.w);
  }
  for (int o = 1; o < 64; o <<= 1) ss += __shfl_xor(ss, o);
  if (lane == 0) ssr[wave] = ss;
  __syncthreads();
  float scale = 1.0f;
  if (p.rms) {
    float q = 0.f;
    for (int w = 0; w < ROWS_WAVES; ++w) q += ssr[w];
    scale = 1.0f / sqrtf(q / (float)p.K + p.eps);
  }
  int par = 0;
  float dummy[1] = {0.f};
  auto use = [&](const uint4* t, int gi, float* acc) {
#pragma unroll
    for (int u = 0; u < GUX; ++u) valu_tile<KPL, 1>(t[u], lo_t + gi * GUX + u, g, xs, p, false, acc, dummy);
  };
  // the finished row block: partial sums of the waves through LDS, then wave 0 alone runs the epilogue on its own
  // LDS patch while the other waves go on with the next row block (the patch is free again by then: wave 0 comes
  // back to it only after the next barrier)
  auto finish = [&](float a, int nb, float res) {
    a += __shfl_xor(a, 16);
    a += __shfl_xor(a, 32);
    if (lane < 16) red[par][wave][lane] = a;
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the partial is in LDS
    __builtin_amdgcn_s_barrier();
    if (wave == 0) {
      if (lane < 16) {
        float s = 0.f;
        for (int w = 0; w < ROWS_WAVES; ++w) s += red[par][w][lane];
        fin[0][lane] = s * scale + res;
      }
      __builtin_amdgcn_wave_barrier();
      epilogue<EPI == EPI_RESID ? EPI_STORE : EPI, true, true>(p, nb, fin, 1, 0, nullptr, nullptr);
      __builtin_amdgcn_wave_barrier();
    }
    par ^= 1;
  };
  // one row block; `more` (fixed per call site): the refills go on into the next row block
  auto block = [&](int nb, bool more) {
    float acc[1] = {0.f};
    // the row block's residual, asked for ahead of its products (by every wave: no branch around a load)
    float res = 0.f;
    if (EPI == EPI_RESID) res = p.R[min(nb * 16 + (lane & 15), p.N - 1)];
    const uint4* wn = wp + blk_stride;
#pragma unroll
    for (int gi = 0; gi < NG; gi += 2) {
      use(ta, gi, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (gi + 2 < NG) fill(ta, wp + (size_t)(gi + 2) * GUX * 64);
      else if (more) fill(ta, wn);
      __builtin_amdgcn_sched_barrier(0);
      use(tb, gi + 1, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (gi + 3 < NG) fill(tb, wp + (size_t)(gi + 3) * GUX * 64);
      else if (more) fill(tb, wn + GUX * 64);
      __builtin_amdgcn_sched_barrier(0);
    }
    finish(acc[0], nb, res);
    wp = wn;
  };
  int nb = wg;
  for (int b = 0; b + 1 < nblk; ++b, nb += nwg) block(nb, true);
  block(nb, false);
}

// ---------------------------------------------------------------------------------------
// Matrix-core skinny GEMM (bf16 weights): out[16 weight rows][16 token rows] per wave via
// v_mfma_f32_16x16x32_bf16, weights as the A operand straight from the tiled layout, token
// rows as the B operand from hi/lo split tiles ([cb][kt][hi|lo][lane][8], lane = 16*(k/8%4) +
// token).  blockIdx.y selects a block of 16 token rows.
// PACK (up to 8 token rows): the high parts are columns 0..7 of the operand and the low parts columns 8..15, so that one
// load and one matrix instruction per weight tile do (against two of each), and column c + 8 is added to column c with
// the waves' partial sums.  What bounds the kernel is how many weight tiles a wave keeps in flight, and the activation
// tiles took two of every three loads.  5 rows, us per launch, separate -> packed: 1376 row blocks of 128 k tiles 33.9 -> 32.8
// (several row blocks per work-group, below), 256 of 344 21.1 -> 20.5, 1728 of 160 52.9 -> 47.3, 320 of 432 40.3 -> 36.7
// (with 8 waves instead of 16), 512 of 896 81.8 -> 77.5; 8 rows gain more (512 of 896: 108 -> 77).
// ---------------------------------------------------------------------------------------
// The piece of a 2 KiB activation tile that a lane supplies; rows beyond the valid ones repeat row 0 (no divergent loads,
// the same cache lines; their columns are never used).
template <bool PACK>
__device__ __forceinline__ int act_piece(int lane, int mvalid) {
  const int c = lane & 15, t = PACK ? c & 7 : c;
  return (PACK && c >= 8 ? 64 : 0) + (lane & 48) + (t < mvalid ? t : 0);
}

template <int EPI, bool PACK>
__global__ void __launch_bounds__(1024) gemm_mfma_k(GemmP p) {
  constexpr int U = 4;
  __shared__ float red[MAXW][16][16];
  __shared__ float fin[16][16];
  __shared__ float scl[16];
  const int tid = threadIdx.x, nw = blockDim.x >> 6, wave = tid >> 6, lane = tid & 63;
  const int nb = blockIdx.x, cb = blockIdx.y;
  const int mvalid = min(16, p.M - cb * 16);
  const int token = lane & 15, g = lane >> 4;
  const int blane = act_piece<PACK>(lane, mvalid);
  int kt_lo, kt_hi;
  wave_span(p.KT, nw, wave, U, kt_lo, kt_hi);
  const int ngroups = (kt_hi - kt_lo) / U;
  const uint4* wp = (const uint4*)p.Wt + ((size_t)nb * p.KT + kt_lo) * 64 + lane;
  const uint4* xp = (const uint4*)p.Xs + ((size_t)cb * p.KT + kt_lo) * 128 + blane;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};   // hi and lo products, independent chains
  // two register sets (even and odd groups), never copied: a copy of a register that a load is still
  // filling would make the wave wait for every load in flight
  uint4 a0[U], h0[U], l0[PACK ? 1 : U], a1[U], h1[U], l1[PACK ? 1 : U];
  auto fill = [&](uint4* a, uint4* bh, uint4* bl, int gi) {
    const uint4* wn = wp + (size_t)gi * U * 64;
    const uint4* xn = xp + (size_t)gi * U * 128;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      a[u] = ld_stream(wn + u * 64);
      bh[u] = xn[u * 128];
      if (!PACK) bl[u] = xn[u * 128 + 64];
    }
  };
  auto use = [&](const uint4* a, const uint4* bh, const uint4* bl) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bf16x8 av = __builtin_bit_cast(bf16x8, a[u]);
      if (PACK) {   // two chains, tiles in turn
        floatx4& c = u & 1 ? acc2 : acc;
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh[u]), c, 0, 0, 0);
      } else {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh[u]), acc, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl[u]), acc2, 0, 0, 0);
      }
    }
  };
  if (ngroups > 0) fill(a0, h0, l0, 0);
  if (ngroups > 1) fill(a1, h1, l1, 1);
  if (p.ssq_in) {   // RMS scale per token row from the producer's per-block sums of squares
    for (int mi = wave; mi < mvalid; mi += nw) {
      float q = 0.f;
      for (int b = lane; b < p.ssq_nb; b += 64) q += p.ssq_in[(size_t)mi * p.ssq_nb + b];
      for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
      if (lane == 0) scl[mi] = 1.0f / sqrtf(q / (float)p.K + p.eps);
    }
  }
  // steady state: branch-free, two groups in flight
  int gi = 0;
  for (; gi + 4 <= ngroups; gi += 2) {
    use(a0, h0, l0);
    fill(a0, h0, l0, gi + 2);
    use(a1, h1, l1);
    fill(a1, h1, l1, gi + 3);
  }
  const int left = ngroups - gi;   // one to three groups, the first two already requested
  if (left == 3) {
    use(a0, h0, l0);
    fill(a0, h0, l0, gi + 2);
    use(a1, h1, l1);
    use(a0, h0, l0);
  } else if (left == 2) {
    use(a0, h0, l0);
    use(a1, h1, l1);
  } else if (left == 1) {
    use(a0, h0, l0);
  }
  for (int kt = kt_lo + ngroups * U; kt < kt_hi; ++kt) {
    const uint4 aw = ld_stream(wp + (size_t)(kt - kt_lo) * 64);
    const uint4 h = xp[(size_t)(kt - kt_lo) * 128];
    const bf16x8 av = __builtin_bit_cast(bf16x8, aw);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, h), acc, 0, 0, 0);
    if (!PACK) {
      const uint4 l = xp[(size_t)(kt - kt_lo) * 128 + 64];
      acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, l), acc2, 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] += acc2[j];
  // D layout: lane holds D[4*(lane/16) + j][lane%16], j = 0..3 (rows = weight rows, cols = tokens)
#pragma unroll
  for (int j = 0; j < 4; ++j) red[wave][token][4 * g + j] = acc[j];
  __syncthreads();
  for (int t = tid; t < 256; t += blockDim.x) {
    const int mi = t >> 4, r = t & 15;
    if (mi < mvalid) {
      float s = 0.f;
      for (int w = 0; w < nw; ++w) s += PACK ? red[w][mi][r] + red[w][mi + 8][r] : red[w][mi][r];
      if (p.rowscale) s *= p.rowscale[cb * 16 + mi];
      if (p.ssq_in) s *= scl[mi];
      fin[mi][r] = s;
    }
  }
  __syncthreads();
  epilogue<EPI, true>(p, nb, fin, mvalid, cb * 16, p.XsOut, p.ssq_out);
}

// ---------------------------------------------------------------------------------------
// The matrix-core skinny GEMM with several row blocks per work-group (up to 16 token rows, KT = 16 * NT: 128 or 160 k
// tiles): as gemv_rows_k, one work-group of 16 waves per compute unit taking the row blocks w, w + grid, ...  A wave
// owns NT k tiles of every row block; the split activation tiles of those k tiles do not depend on the row block, so
// they are loaded once and stay in registers for all of the work-group's row blocks (the form above fetches them again
// with every weight tile).  Weight tiles: two named sets of HS, refilled as soon as used, running on into the next row
// block; 16 waves per work-group cap a wave at 128 registers, so that with separate high and low parts (more than 8
// token rows) only NT = 8 fits, with sets of 2; packed, a tile is 4 registers and the sets are as deep as the one-row
// kernel's.  Wave 0 sums the waves' 16x16 partials and runs the epilogue while the others go on.
// ---------------------------------------------------------------------------------------
template <int EPI, bool PACK, int NT, int HS>
__global__ void __launch_bounds__(1024) gemm_mfma_rows_k(GemmP p) {
  static_assert(NT % (2 * HS) == 0, "the two sets take the tiles in turn");
  __shared__ float red[2][ROWS_WAVES][16][16];
  __shared__ float fin[16][16];
  __shared__ float scl[16];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wg = blockIdx.x, nwg = gridDim.x;
  if (wg >= p.NB) return;                                // uniform, before any barrier
  const int nblk = (p.NB - wg + nwg - 1) / nwg;
  const int KT = p.KT;                                   // = 16 * NT
  const int mvalid = min(16, p.M);
  const int token = lane & 15, g = lane >> 4;
  const int blane = act_piece<PACK>(lane, mvalid);
  const int lo_t = wave * NT;
  // this wave's activation tiles for its k tiles: loaded once
  uint4 bh[NT], bl[PACK ? 1 : NT];
  const uint4* xp = (const uint4*)p.Xs + (size_t)lo_t * 128 + blane;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    bh[i] = xp[i * 128];
    if (!PACK) bl[i] = xp[i * 128 + 64];
  }
  const size_t blk_stride = (size_t)nwg * KT * 64;
  const uint4* wp = (const uint4*)p.Wt + ((size_t)wg * KT + lo_t) * 64 + lane;
  uint4 ta[HS], tb[HS];
  auto fill = [&](uint4* t, const uint4* src) {
#pragma unroll
    for (int u = 0; u < HS; ++u) t[u] = ld_stream(src + u * 64);
  };
  fill(ta, wp);
  fill(tb, wp + HS * 64);
  if (p.ssq_in) {   // RMS scale per token row from the producer's per-block sums of squares
    for (int mi = wave; mi < mvalid; mi += ROWS_WAVES) {
      float q = 0.f;
      for (int b = lane; b < p.ssq_nb; b += 64) q += p.ssq_in[(size_t)mi * p.ssq_nb + b];
      for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
      if (lane == 0) scl[mi] = 1.0f / sqrtf(q / (float)p.K + p.eps);
    }
  }
  __syncthreads();
  int par = 0;
  auto finish = [&](const floatx4& acc, int nb) {
    // D layout: lane holds D[4*(lane/16) + j][lane%16], j = 0..3 (rows = weight rows, cols = tokens)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[par][wave][token][4 * g + j] = acc[j];
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = lane + 64 * i, mi = t >> 4, r = t & 15;
        if (mi < mvalid) {
          float s = 0.f;
          for (int w = 0; w < ROWS_WAVES; ++w) s += PACK ? red[par][w][mi][r] + red[par][w][mi + 8][r] : red[par][w][mi][r];
          if (p.rowscale) s *= p.rowscale[mi];
          if (p.ssq_in) s *= scl[mi];
          fin[mi][r] = s;
        }
      }
      __builtin_amdgcn_wave_barrier();
      epilogue<EPI, true, true>(p, nb, fin, mvalid, 0, p.XsOut, p.ssq_out);
      __builtin_amdgcn_wave_barrier();
    }
    par ^= 1;
  };
  auto block = [&](int nb, bool more) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    const uint4* wn = wp + blk_stride;
    auto use = [&](const uint4* t, int i0) {
#pragma unroll
      for (int u = 0; u < HS; ++u) {
        const bf16x8 av = __builtin_bit_cast(bf16x8, t[u]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh[i0 + u]), acc, 0, 0, 0);
        if (!PACK) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl[i0 + u]), acc, 0, 0, 0);
      }
    };
#pragma unroll
    for (int i0 = 0; i0 < NT; i0 += 2 * HS) {
      use(ta, i0);
      __builtin_amdgcn_sched_barrier(0);
      if (i0 + 2 * HS < NT) fill(ta, wp + (size_t)(i0 + 2 * HS) * 64);
      else if (more) fill(ta, wn);
      __builtin_amdgcn_sched_barrier(0);
      use(tb, i0 + HS);
      __builtin_amdgcn_sched_barrier(0);
      if (i0 + 3 * HS < NT) fill(tb, wp + (size_t)(i0 + 3 * HS) * 64);
      else if (more) fill(tb, wn + HS * 64);
      __builtin_amdgcn_sched_barrier(0);
    }
    finish(acc, nb);
    wp = wn;
  };
  int nb = wg;
  for (int b = 0; b + 1 < nblk; ++b, nb += nwg) block(nb, true);
  block(nb, false);
}

// ---------------------------------------------------------------------------------------
// fp32 rows -> bf16 hi/lo split tiles (+ optional gain and inverse RMS per row).
// One work-group per row; a thread takes eight features at a time (two 16-byte loads, two 16-byte stores; element by
// element with a second pass for the sum of squares the 8 to 512 rows of a shadow head took 11 to 18 us).
// Rows are padded to whole k tiles, and so is the gain.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) prep_split_k(const float* src, int rows_per_group, long long group_stride,
                                                    int ld, int K, int KT, const float* gain, int rms, float eps,
                                                    uint16_t* Xs, float* rowscale) {
  __shared__ float part[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const int grp = row / rows_per_group, i = row - grp * rows_per_group;
  const float* x = src + (size_t)grp * group_stride + (size_t)i * ld;
  const int cb = row >> 4, token = row & 15;
  uint16_t* out = Xs + (size_t)cb * KT * 1024;
  float ss = 0.f;
  for (int c = tid; c < KT * 4; c += 256) {
    const int k = c * 8;
    const float4 a = *(const float4*)(x + k), b = *(const float4*)(x + k + 4);
    float4 g0 = make_float4(1.f, 1.f, 1.f, 1.f), g1 = g0;
    if (gain) { g0 = *(const float4*)(gain + k); g1 = *(const float4*)(gain + k + 4); }
    float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (k + e >= K) v[e] = 0.f;
      ss += v[e] * v[e];
      v[e] *= g[e];
    }
    split_store8(out, c, token, v);
  }
  if (!rms) {
    if (tid == 0) rowscale[row] = 1.0f;
    return;
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) rowscale[row] = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)K + eps);
}

// ---------------------------------------------------------------------------------------
// Attention over the KV cache, split over the context: one work-group per (chunk of p.ct cache
// rows, kv head).  K and V of the chunk are fetched with all loads in flight at once, staged
// in LDS and shared by every query row of the head group (m token rows x n_q/n_kv heads).
// Emits softmax partials (max, sum, weighted values); attn_combine_k merges the chunks.
// Caches are [n_kv][Tcap][hd].
// ---------------------------------------------------------------------------------------
template <typename KVT>
__global__ void __launch_bounds__(256) attn_partial_k(AttnP p) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int EPW = 4 / sizeof(KVT);  // elements per 32-bit word
  constexpr int NLD = 4;                // 16-byte loads per thread and matrix (64 rows x 256 B at most)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = blockIdx.x, kvh = blockIdx.y;
  const int ct = p.ct;
  const int T0 = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off;
  const int T_end = T0 + p.m;
  const int t0 = c * ct;
  if (t0 >= T_end) return;
  const int nt = min(ct, T_end - t0);
  const int hd = p.hd, G = p.n_q / p.n_kv, QR = p.m * G;
  const int QB = p.qb;        // query rows per batch (LDS is sized for it)
  const int wpr = hd / EPW;   // words per cache row
  const int ksw = wpr + 1;    // padded LDS row stride in words
  const int rb16 = wpr >> 2;  // 16-byte pieces per cache row
  uint32_t* Ks = (uint32_t*)smem;
  uint32_t* Vs = Ks + ct * ksw;
  float* Qs = (float*)(Vs + ct * ksw);
  float* Ss = Qs + QB * hd;
  const uint4* Kg = (const uint4*)((const KVT*)p.Kc + ((size_t)kvh * p.Tcap + t0) * hd);
  const uint4* Vg = (const uint4*)((const KVT*)p.Vc + ((size_t)kvh * p.Tcap + t0) * hd);
  const int npieces = nt * rb16;
  const float scale = 1.0f / sqrtf((float)hd);
  // few query rows (decode): fetch them now, together with K and V
  const bool qfast = QR * hd <= 4 * 256;
  float qreg[4];
  if (qfast) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = tid + 256 * j;
      qreg[j] = 0.f;
      if (i < QR * hd) {
        const int qi = i / hd, d = i - qi * hd;
        const int mi = qi / G, gi = qi - mi * G;
        qreg[j] = p.Q[(size_t)mi * p.ldq + (kvh * G + gi) * hd + d] * scale;
      }
    }
  }
  uint4 kr[NLD], vr[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int i = tid + 256 * j;
    kr[j] = vr[j] = make_uint4(0, 0, 0, 0);
    if (i < npieces) { kr[j] = Kg[i]; vr[j] = Vg[i]; }
  }
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int i = tid + 256 * j;
    if (i < npieces) {
      const int row = i / rb16, w = (i - row * rb16) * 4;
      uint32_t* kd = Ks + row * ksw + w;
      uint32_t* vd = Vs + row * ksw + w;
      kd[0] = kr[j].x; kd[1] = kr[j].y; kd[2] = kr[j].z; kd[3] = kr[j].w;
      vd[0] = vr[j].x; vd[1] = vr[j].y; vd[2] = vr[j].z; vd[3] = vr[j].w;
    }
  }
  if (qfast) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = tid + 256 * j;
      if (i < QR * hd) Qs[i] = qreg[j];
    }
  }
  const int dpairs = hd >> 1;          // PV step: one thread per pair of value dims
  const int nslots = 256 / dpairs;     // query rows processed side by side in the PV step
  const int d2 = tid % dpairs, qslot = tid / dpairs;
  for (int qb = 0; qb < QR; qb += QB) {
    const int nq = min(QB, QR - qb);
    if (!qfast) {
      __syncthreads();
      for (int i = tid; i < nq * hd; i += 256) {
        const int qi = i / hd, d = i - qi * hd;
        const int qr = qb + qi, mi = qr / G, gi = qr - mi * G;
        Qs[qi * hd + d] = p.Q[(size_t)mi * p.ldq + (kvh * G + gi) * hd + d] * scale;
      }
    }
    __syncthreads();
    // scores: one (query row, cache row) pair per thread and step
    for (int pi = tid; pi < nq * ct; pi += 256) {
      const int qi = pi / ct, t = pi - qi * ct;
      const int mi = (qb + qi) / G;
      float s = -INFINITY;
      if (t < nt && t0 + t <= T0 + mi) {
        const uint32_t* krow = Ks + t * ksw;
        const float* qv = Qs + qi * hd;
        float a = 0.f;
        if (sizeof(KVT) == 2) {
          for (int w = 0; w < wpr; ++w) {
            const uint32_t kk = krow[w];
            a += qv[2 * w] * __uint_as_float(kk << 16);
            a += qv[2 * w + 1] * __uint_as_float(kk & 0xFFFF0000u);
          }
        } else {
          for (int w = 0; w < wpr; ++w) a += qv[w] * __uint_as_float(krow[w]);
        }
        s = a;
      }
      Ss[qi * ct + t] = s;
    }
    __syncthreads();
    // softmax numerators per row: one wave per query row, lanes over the cache rows
    for (int qi = wave; qi < nq; qi += 4) {
      float sv = lane < ct ? Ss[qi * ct + lane] : -INFINITY;
      float mx = sv;
      for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
      const float pr = mx > -INFINITY ? expf(sv - mx) : 0.f;   // masked entries: exp(-inf) = 0
      float l = pr;
      for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
      if (lane < ct) Ss[qi * ct + lane] = pr;
      if (lane == 0) {
        const int qr = qb + qi, mi = qr / G, gi = qr - mi * G;
        const size_t prow = ((size_t)mi * p.n_q + kvh * G + gi) * p.nch_max + c;
        p.PM[prow] = mx;
        p.PL[prow] = l;
      }
    }
    __syncthreads();
    // weighted values
    for (int qi = qslot < nslots ? qslot : nq; qi < nq; qi += nslots) {
      const float* pr = Ss + qi * ct;
      float a0 = 0.f, a1 = 0.f;
      if (sizeof(KVT) == 2) {
        const uint32_t* vcol = Vs + d2;
        for (int t = 0; t < nt; ++t) {
          const uint32_t vv = vcol[t * ksw];
          a0 += pr[t] * __uint_as_float(vv << 16);
          a1 += pr[t] * __uint_as_float(vv & 0xFFFF0000u);
        }
      } else {
        const uint32_t* vcol = Vs + 2 * d2;
        for (int t = 0; t < nt; ++t) {
          a0 += pr[t] * __uint_as_float(vcol[t * ksw]);
          a1 += pr[t] * __uint_as_float(vcol[t * ksw + 1]);
        }
      }
      const int qr = qb + qi, mi = qr / G, gi = qr - mi * G;
      const size_t prow = ((size_t)mi * p.n_q + kvh * G + gi) * p.nch_max + c;
      *(float2*)(p.PA + prow * hd + 2 * d2) = make_float2(a0, a1);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Decode attention (one new token row): one work-group per (split of the context, kv head),
// 8 waves.  A wave-wide 16-byte load covers 64/LPR whole cache rows (LPR lanes per row); each
// lane keeps its slice of q in registers, scores are reduced over the LPR lanes of a row, and
// every lane group runs its own online softmax over the rows it sees, so K and V go from HBM
// to registers once with eight 1 KiB loads in flight per wave.  Lane groups and waves are
// merged at the end; the S per-split partials are merged by the consumer (the O projection's
// input staging), so no combine kernel runs on this path.
// ---------------------------------------------------------------------------------------
struct SoftAcc { float m, l; };

// RW > 1 (prefill): RW consecutive token rows share the work-group's cache reads; query q = r * G + g
// is head g of the kv group for token row mi0 + r and sees cache rows up to its own position only.
template <typename KVT, int HD, int G, int RW>
__global__ void __launch_bounds__(512) attn_decode_k(AttnP p) {
  constexpr int NQ = G * RW;
  constexpr int EPL = 16 / sizeof(KVT);   // elements per lane and load
  constexpr int LPR = HD / EPL;           // lanes per cache row
  constexpr int RPL = 64 / LPR;           // cache rows per wave-wide load
  constexpr int UL = 4;                   // loads in flight per wave, matrix and pipeline stage
  constexpr int NWV = RW > 1 ? 4 : 8;           // waves per work-group (launched with 64 * NWV threads)
  __shared__ float sm[NWV][NQ], sl[NWV][NQ];
  __shared__ float sa[NWV][NQ][HD];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int split = blockIdx.x, kvh = blockIdx.y, S = gridDim.x;
  const int mi0 = blockIdx.z * RW;                        // first token row of this work-group
  const int nrow = min(RW, p.m - mi0);                    // rows it really has
  const int T0 = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off + mi0;   // row mi0 + r attends cache rows <= T0 + r
  const int T_end = T0 + nrow;
  const int rps = ((T_end + S - 1) / S + RPL - 1) / RPL * RPL;   // rows per split, whole loads
  const int t_lo = split * rps, t_hi = min(T_end, t_lo + rps);
  const int rs = lane / LPR, dl = lane % LPR;
  const float scale = 1.0f / sqrtf((float)HD);
  float q[NQ][EPL];
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    // a ragged last group re-reads its last row; those queries' results are dropped
    const float* qp = p.Q + (size_t)(mi0 + min(g / G, nrow - 1)) * p.ldq + (size_t)(kvh * G + g % G) * HD + dl * EPL;
#pragma unroll
    for (int e = 0; e < EPL; e += 4) {
      const float4 t = *(const float4*)(qp + e);
      q[g][e] = t.x * scale; q[g][e + 1] = t.y * scale; q[g][e + 2] = t.z * scale; q[g][e + 3] = t.w * scale;
    }
  }
  float m[NQ], l[NQ], acc[NQ][EPL];
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
    m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.f;
  }
  // row groups of this wave: j = wave, wave + NWV, ...; group j covers rows t_lo + j*RPL ...
  const int ngrp = t_hi > t_lo ? (t_hi - t_lo + RPL - 1) / RPL : 0;
  const uint4* Kg = (const uint4*)((const KVT*)p.Kc + (size_t)kvh * p.Tcap * HD);
  const uint4* Vg = (const uint4*)((const KVT*)p.Vc + (size_t)kvh * p.Tcap * HD);
  // rows past t_hi (a ragged last group) are read from row t_hi - 1 and masked
  auto row_of = [&](int j) { return min(t_lo + j * RPL + rs, t_hi - 1); };
  uint4 kc[UL], vc[UL], kn[UL], vn[UL];
  auto consume = [&](const uint4& kk, const uint4& vv, int j) {
    const int trow = t_lo + j * RPL + rs;
    const bool valid = j < ngrp && trow < t_hi;
    float kf[EPL], vf[EPL];
    if (sizeof(KVT) == 2) { WDec<8>::dec(kk, kf); WDec<8>::dec(vv, vf); }
    else { WDec<4>::dec(kk, kf); WDec<4>::dec(vv, vf); }
#pragma unroll
    for (int g = 0; g < NQ; ++g) {
      float sdot = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) sdot += q[g][e] * kf[e];
#pragma unroll
      for (int o = 1; o < LPR; o <<= 1) sdot += __shfl_xor(sdot, o);
      if (valid && (RW == 1 || trow <= T0 + g / G)) {
        const float mn = fmaxf(m[g], sdot);
        const float c = expf(m[g] - mn);      // m = -inf at the first row: exp(-inf) = 0
        const float pr = expf(sdot - mn);
        l[g] = l[g] * c + pr;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = acc[g][e] * c + pr * vf[e];
        m[g] = mn;
      }
    }
  };
  if (ngrp > 0) {
    const int nit = (ngrp - wave + NWV * UL - 1) / (NWV * UL);   // iterations of this wave (may be <= 0)
    if (nit > 0) {
#pragma unroll
      for (int u = 0; u < UL; ++u) {
        const int j = min(wave + u * NWV, ngrp - 1);
        const size_t off = (size_t)row_of(j) * LPR + dl;
        kc[u] = Kg[off]; vc[u] = Vg[off];
      }
      for (int it = 0; it < nit; ++it) {
        const int j0 = wave + it * NWV * UL;
#pragma unroll
        for (int u = 0; u < UL; ++u) {   // next iteration's rows (clamped: re-reads the last group at the end)
          const int j = min(j0 + (UL + u) * NWV, ngrp - 1);
          const size_t off = (size_t)row_of(j) * LPR + dl;
          kn[u] = Kg[off]; vn[u] = Vg[off];
        }
#pragma unroll
        for (int u = 0; u < UL; ++u) consume(kc[u], vc[u], j0 + u * NWV);
#pragma unroll
        for (int u = 0; u < UL; ++u) { kc[u] = kn[u]; vc[u] = vn[u]; }
      }
    }
  }
  // merge the lane groups of a wave (same value dims, different rows) ...
#pragma unroll
  for (int g = 0; g < NQ; ++g) {
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      const float m2 = __shfl_xor(m[g], o), l2 = __shfl_xor(l[g], o);
      const float M = fmaxf(m[g], m2);
      const float c1 = m[g] > -INFINITY ? expf(m[g] - M) : 0.f;
      const float c2 = m2 > -INFINITY ? expf(m2 - M) : 0.f;
      l[g] = l[g] * c1 + l2 * c2;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] = acc[g][e] * c1 + __shfl_xor(acc[g][e], o) * c2;
      m[g] = M;
    }
    if (rs == 0) {
      if (dl == 0) { sm[wave][g] = m[g]; sl[wave][g] = l[g]; }
#pragma unroll
      for (int e = 0; e < EPL; ++e) sa[wave][g][dl * EPL + e] = acc[g][e];
    }
  }
  __syncthreads();
  // ... then the waves, in a fixed order; one partial per (query row, split)
  for (int i = tid; i < NQ * HD; i += 64 * NWV) {
    const int g = i / HD, d = i - g * HD;
    if (g / G >= nrow) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NWV; ++w) M = fmaxf(M, sm[w][g]);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      const float c = sm[w][g] > -INFINITY ? expf(sm[w][g] - M) : 0.f;
      L += c * sl[w][g];
      A += c * sa[w][g][d];
    }
    const int mi = mi0 + g / G, h = kvh * G + g % G;
    if (S == 1 && p.nsplit < 0) {
      // a single split and the caller wants the result itself: output row and its split tile, no partials
      const float o = A / L;
      p.O[(size_t)mi * p.ldo + h * HD + d] = o;
      if (p.XsOut) {
        const int k = h * HD + d;
        const uint16_t hi = f32_to_bf16_rne(o);
        const uint16_t lo = f32_to_bf16_rne(o - bf16_bits_to_f32(hi));
        uint16_t* dst = p.XsOut + (size_t)(mi >> 4) * p.xs_cb_stride + (size_t)(k >> 5) * 1024 +
                        (((k & 31) >> 3) * 16 + (mi & 15)) * 8 + (k & 7);
        dst[0] = hi;
        dst[512] = lo;
      }
      continue;
    }
    const size_t prow = ((size_t)mi * p.n_q + h) * p.nch_max + split;
    if (d == 0) { p.PM[prow] = M; p.PL[prow] = L; }
    p.PA[prow * HD + d] = A;
  }
}

__device__ __forceinline__ void split8(const float* v, uint4& hi, uint4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const uint16_t h0 = f32_to_bf16_rne(v[e]), h1 = f32_to_bf16_rne(v[e + 1]);
    const uint16_t l0 = f32_to_bf16_rne(v[e] - bf16_bits_to_f32(h0));
    const uint16_t l1 = f32_to_bf16_rne(v[e + 1] - bf16_bits_to_f32(h1));
    h[e >> 1] = (uint32_t)h0 | ((uint32_t)h1 << 16);
    l[e >> 1] = (uint32_t)l0 | ((uint32_t)l1 << 16);
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// ---------------------------------------------------------------------------------------
// Matrix-core attention for a few token rows (the verify pass: m <= 16 rows, Section 2 "verifies all draft tokens in
// parallel"), split over the context: one wave = all m queries of one query head against one span of cache rows, so
// the cache is read once for all rows and there are (splits x query heads) waves to keep in flight.  Each wave leaves
// a soft-max partial (max, sum, weighted values) per (token row, head, split); attn_combine_k merges them.  Per 32
// cache rows:
//   S^T[32 rows][16 queries] = K[32][hd] * Q^T      (A = cache rows as stored, B = queries as
//                                                    bf16 high + low parts, kept in registers)
//   online soft-max per query (a lane holds 8 rows of one query; two cross-lane steps)
//   O^T[hd][16 queries] += V^T[hd][32 rows] * P     (A = the feature-major copy of the values,
//                                                    B = the probabilities, high + low parts)
// The A operand of the first product takes cache row t0 + 8*(i/4) + i%4 (+4 for the second block
// of 16) as its row i, so that the 8 scores a lane ends up with are 8 consecutive cache rows:
// exactly the B operand slice it must supply to the second product.  Nothing passes through LDS.
// ---------------------------------------------------------------------------------------
template <int HD>
__global__ void __launch_bounds__(256) attn_flash_split_k(AttnP p, int S, int rps_min) {
  constexpr int KT = HD / 32, DT = HD / 16;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, qi = lane & 15;
  const int split = blockIdx.x * 4 + wave;
  if (split >= S) return;                      // wave-uniform; the kernel has no barriers
  const int h = blockIdx.y, kvh = h / (p.n_q / p.n_kv);
  const int nrow = p.m;                        // <= 16, checked by the launcher
  const int T0 = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off;       // cache position of token row 0
  const int pos = T0 + qi;                     // this lane's query attends cache rows <= pos
  const int t_end = T0 + nrow;                 // cache rows the pass needs: [0, t_end)
  // rows per split: whole tiles of 32, at least what the launcher planned for (attn_combine_k derives the
  // same number from p.rps)
  const int rps = max(rps_min, ((t_end + S - 1) / S + 31) / 32 * 32);
  const int t_lo = split * rps, t_hi = min(t_end, t_lo + rps);
  if (t_lo >= t_end) return;                   // a span past the context: the merge does not read its partial
  uint4 qh[KT], ql[KT];
  {
    const float scale = 1.0f / sqrtf((float)HD);
    const float* qp = p.Q + (size_t)min(qi, nrow - 1) * p.ldq + (size_t)h * HD + 8 * g;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const float4 a = *(const float4*)(qp + 32 * kt), b = *(const float4*)(qp + 32 * kt + 4);
      const float v[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale,
                          b.x * scale, b.y * scale, b.z * scale, b.w * scale};
      split8(v, qh[kt], ql[kt]);
    }
  }
  floatx4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = (floatx4){0.f, 0.f, 0.f, 0.f};
  float mrun = -INFINITY, lrun = 0.f;
  const uint16_t* Kb = (const uint16_t*)p.Kc + (size_t)kvh * p.Tcap * HD + 8 * g;
  const uint16_t* Vt = (const uint16_t*)p.VcT + ((size_t)kvh * HD + qi) * p.TcapT + 8 * g;
  const int rho = 8 * (qi >> 2) + (qi & 3);
  // two register sets, filled and used in turn: the rows of the next tile are requested before the current
  // tile is multiplied (a span is two or three tiles: without this each tile costs a full memory latency).
  // Branch-free: an odd tile count runs one more, fully masked, tile on a re-read of the last one.
  auto load = [&](int t0, uint4* a0, uint4* a1, uint4* av) {
    // rows past the pass's last one are read from that last row and masked in the scores
    const uint16_t* k0 = Kb + (size_t)min(t0 + rho, t_end - 1) * HD;
    const uint16_t* k1 = Kb + (size_t)min(t0 + rho + 4, t_end - 1) * HD;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      a0[kt] = *(const uint4*)(k0 + 32 * kt);
      a1[kt] = *(const uint4*)(k1 + 32 * kt);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) av[dt] = *(const uint4*)(Vt + (size_t)(16 * dt) * p.TcapT + t0);
  };
  auto compute = [&](int t0, const uint4* a0, const uint4* a1, const uint4* av) {
    floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const bf16x8 x0 = __builtin_bit_cast(bf16x8, a0[kt]), x1 = __builtin_bit_cast(bf16x8, a1[kt]);
      const bf16x8 bh = __builtin_bit_cast(bf16x8, qh[kt]), bl = __builtin_bit_cast(bf16x8, ql[kt]);
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, bh, s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, bh, s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, bl, s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, bl, s1, 0, 0, 0);
    }
    // this lane: scores of cache rows t0 + 8g + e, e = 0..7, for query qi; rows of the next span (the extra
    // tile of an odd count) and rows the query may not see count for nothing
    float sv[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int row = t0 + 8 * g + e;
      if (row > pos || row >= t_hi) sv[e] = -INFINITY;
      mx = fmaxf(mx, sv[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // a split may hold no row this query may see (the rows of later tokens only): everything stays
    // at (max = -inf, sum = 0, values = 0), which the merge gives weight 0
    const float mnew = fmaxf(mrun, mx);
    const float c = mrun > -INFINITY ? expf(mrun - mnew) : 0.f;
    float pv[8], ls = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pv[e] = sv[e] > -INFINITY ? expf(sv[e] - mnew) : 0.f;
      ls += pv[e];
    }
    ls += __shfl_xor(ls, 16);
    ls += __shfl_xor(ls, 32);
    lrun = lrun * c + ls;
    mrun = mnew;
    uint4 ph, pl;
    split8(pv, ph, pl);
    const bf16x8 bh = __builtin_bit_cast(bf16x8, ph), bl = __builtin_bit_cast(bf16x8, pl);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int j = 0; j < 4; ++j) o[dt][j] *= c;
      const bf16x8 x = __builtin_bit_cast(bf16x8, av[dt]);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, bh, o[dt], 0, 0, 0);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, bl, o[dt], 0, 0, 0);
    }
  };
  {
    const int last = t_lo + (t_hi - t_lo - 1) / 32 * 32;   // first row of the span's last tile
    uint4 ka0[KT], ka1[KT], va[DT], kb0[KT], kb1[KT], vb[DT];
    load(t_lo, ka0, ka1, va);
    for (int t0 = t_lo; t0 < t_hi; t0 += 64) {
      load(min(t0 + 32, last), kb0, kb1, vb);
      compute(t0, ka0, ka1, va);
      load(min(t0 + 64, last), ka0, ka1, va);
      compute(t0 + 32, kb0, kb1, vb);
    }
  }
  if (qi >= nrow) return;
  // this lane: features 16*dt + 4g + j of head h for token row qi, as an unnormalised partial
  const size_t prow = ((size_t)qi * p.n_q + h) * p.nch_max + split;
  if (g == 0) { p.PM[prow] = mrun; p.PL[prow] = lrun; }
  float* pa = p.PA + prow * HD + 4 * g;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) *(float4*)(pa + 16 * dt) = make_float4(o[dt][0], o[dt][1], o[dt][2], o[dt][3]);
}

__global__ void __launch_bounds__(128) attn_combine_k(AttnP p) {
  const int row = blockIdx.x;  // mi * n_q + h
  const int d = threadIdx.x;
  if (d >= p.hd) return;
  const int T_end = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off + p.m;
  int nch = p.nsplit > 0 ? p.nsplit : (T_end + p.ct - 1) / p.ct;   // partials per row
  if (p.rps > 0) {   // matrix-core kernel, split by spans of rows: only the spans that reach into the context
    const int rps = max(p.rps, ((T_end + p.nsplit - 1) / p.nsplit + 31) / 32 * 32);
    nch = min(nch, (T_end + rps - 1) / rps);
  }
  const float* pm = p.PM + (size_t)row * p.nch_max;
  const float* pl = p.PL + (size_t)row * p.nch_max;
  const float* pa = p.PA + (size_t)row * p.nch_max * p.hd + d;
  // every chunk below nch has written its partial (fully masked ones: max = -inf, sum = 0, values = 0),
  // so the loops are branch-free and their loads independent
  float M = -INFINITY;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) M = fmaxf(M, pm[c]);
  float L = 0.f, acc = 0.f;
#pragma unroll 8
  for (int c = 0; c < nch; ++c) {
    const float mc = pm[c];
    const float w = mc > -INFINITY ? expf(mc - M) : 0.f;
    L += w * pl[c];
    acc += w * pa[(size_t)c * p.hd];
  }
  const int mi = row / p.n_q, h = row - mi * p.n_q;
  const float o = acc / L;
  p.O[(size_t)mi * p.ldo + h * p.hd + d] = o;
  if (p.XsOut) {
    const int k = h * p.hd + d;
    const uint16_t hi = f32_to_bf16_rne(o);
    const uint16_t lo = f32_to_bf16_rne(o - bf16_bits_to_f32(hi));
    uint16_t* dst = p.XsOut + (size_t)(mi >> 4) * p.xs_cb_stride + (size_t)(k >> 5) * 1024 +
                    (((k & 31) >> 3) * 16 + (mi & 15)) * 8 + (k & 7);
    dst[0] = hi;
    dst[512] = lo;
  }
}

// ---------------------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------------------
template <int KPL>
__global__ void __launch_bounds__(256) embed_k(const void* Et, int KT, int vocab, const int* ids, float* out, int ld,
                                               int d_model) {
  const int row = blockIdx.x;
  int id = ids[row];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
  gather_embedding(Et, KPL, KT, id, out + (size_t)row * ld, d_model, threadIdx.x, 256);
}

// Merge the per-row-block (max, index) partials of one logits row; lowest index wins ties.
// With psum (per-block sums of exp(logit - block max)) also the confidence of the arg-max token:
// its soft-max probability 1 / sum_b psum[b] * exp(max_b - max) (Section 4.4).
// emb_out (optional, one row): the winner's embedding row goes there as fp32 (the next draft step's input),
// read from the tiled embedding Et (kpl = 8 bf16 or 4 fp32 elements per lane and tile).
// Bound by memory latency, one round trip per batch of loads: a thread asks for AF_UN partials of all three arrays at
// once (one at a time, in a second pass for the sums, 8016 partials took 22 us).
constexpr int AF_UN = 8;
__global__ void __launch_bounds__(1024) argmax_finish_k(const float* pval, const int* pidx, const float* psum, int NB,
                                                        int* out_ids, float* out_conf, const void* Et, int kpl,
                                                        int KT_e, int vocab, float* emb_out, int d_model,
                                                        unsigned long long* note, unsigned seq) {
  __shared__ float sv[MAXW], sw[MAXW];
  __shared__ int si[MAXW];
  const int row = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x, wave = tid >> 6, nw = nthr >> 6;
  const float* pv = pval + (size_t)row * NB;
  const int* pi = pidx + (size_t)row * NB;
  const bool conf = psum && out_conf;
  const float* ps = conf ? psum + (size_t)row * NB : pv;   // (unused values where there is no confidence)
  float best = -INFINITY, se = 0.f;                        // se: relative to best
  int bi = 0x7FFFFFFF;
  for (int b0 = tid; b0 < NB; b0 += AF_UN * nthr) {
    float v[AF_UN], w[AF_UN];
    int ix[AF_UN];
#pragma unroll
    for (int u = 0; u < AF_UN; ++u) {
      const int b = min(b0 + u * nthr, NB - 1);
      v[u] = pv[b]; ix[u] = pi[b]; w[u] = ps[b];
    }
    const float before = best;
#pragma unroll
    for (int u = 0; u < AF_UN; ++u) {
      if (b0 + u * nthr >= NB) v[u] = -INFINITY;
      if (v[u] > best || (v[u] == best && ix[u] < bi && b0 + u * nthr < NB)) { best = v[u]; bi = ix[u]; }
    }
    if (conf) {
      se = before > -INFINITY ? se * expf(before - best) : 0.f;
#pragma unroll
      for (int u = 0; u < AF_UN; ++u)
        if (v[u] > -INFINITY) se += w[u] * expf(v[u] - best);
    }
  }
  const float mine = best;
  for (int o = 32; o > 0; o >>= 1) {
    const float v = __shfl_xor(best, o);
    const int ix = __shfl_xor(bi, o);
    if (v > best || (v == best && ix < bi)) { best = v; bi = ix; }
  }
  if ((tid & 63) == 0) { sv[wave] = best; si[wave] = bi; }
  __syncthreads();
  float M = sv[0];
  int winner = si[0];
  for (int w = 1; w < nw; ++w)
    if (sv[w] > M || (sv[w] == M && si[w] < winner)) { M = sv[w]; winner = si[w]; }
  if (tid == 0) out_ids[row] = winner;
  if (emb_out && row == 0) {
    const int id = winner < 0 ? 0 : (winner >= vocab ? vocab - 1 : winner);
    gather_embedding(Et, kpl, KT_e, id, emb_out, d_model, tid, nthr);
  }
  if (conf) {
    se = mine > -INFINITY ? se * expf(mine - M) : 0.f;
    for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
    if ((tid & 63) == 0) sw[wave] = se;
    __syncthreads();
    if (tid == 0) {
      float sum = 0.f;
      for (int w = 0; w < nw; ++w) sum += sw[w];
      const float cf = 1.0f / sum;
      out_conf[row] = cf;
      // for a host that polls pinned memory instead of waiting for the stream: sequence number and
      // confidence in one 8-byte store
      if (note && row == 0)
        __hip_atomic_store(note, ((unsigned long long)seq << 32) | __float_as_uint(cf), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// Greedy acceptance on the device (Section 2, greedy special case): u = first i < gamma
// with draft[i] != target[i], else gamma; the KV length advances by u + 1 and the pending
// input token becomes the target's token at u.  The drafted tokens are layer E's shadow
// tokens by construction, so they overwrite that row (both were computed from the same
// hidden state, but by different kernels).
// result: [0]=u, [1]=new T, [2]=pending, [3..3+gamma) drafts, then shadow [L][m]
__global__ void accept_k(int* state, const int* draft_ids, int* shadow_ids, int L, int m, int E, int gamma,
                         int* result) {
  // one wave: the drafts stand in for layer E's shadow tokens, then the first mismatch, then the copies
  const int t = threadIdx.x;
  if (blockIdx.x != 0 || t >= 64) return;
  int* srow = shadow_ids + (size_t)(E - 1) * m;
  for (int i = t; i < gamma; i += 64) srow[i] = draft_ids[i];
  const int* target = shadow_ids + (size_t)(L - 1) * m;
  // lane i < gamma looks at draft i (gamma <= 64 is checked by the launcher)
  const bool miss = t < gamma && draft_ids[t] != target[t];
  const unsigned long long mm = __ballot(miss);
  const int u = mm ? __ffsll((long long)mm) - 1 : gamma;
  const int T = state[0] + u + 1;
  const int next = target[u];
  __builtin_amdgcn_wave_barrier();
  if (t == 0) {
    state[0] = T;
    state[1] = next;
    result[0] = u;
    result[1] = T;
    result[2] = next;
  }
  for (int i = t; i < gamma; i += 64) result[3 + i] = draft_ids[i];
  // layer E's row was rewritten above by this same wave; its stores precede these loads in program order
  __threadfence_block();
  for (int i = t; i < L * m; i += 64) result[3 + gamma + i] = shadow_ids[i];
}

__global__ void set_state_k(int* state, int add_T, int set_T, const int* pending_src, int pending_val) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (set_T >= 0) state[0] = set_T;
  state[0] += add_T;
  if (pending_src) state[1] = *pending_src;
  else if (pending_val >= 0) state[1] = pending_val;
}

// Natural row-major [nrows, cols] (rows row0.. of the tensor) -> tiled layout, with the row map.
template <int KPL, typename T>
__global__ void __launch_bounds__(256) tile_scatter_k(const T* src, long long row0, long long nrows, long long cols,
                                                      int map, int vbase, int hd, T* dst, int KT) {
  const long long chunks_per_row = (cols + KPL - 1) / KPL;
  const long long total = nrows * chunks_per_row;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const long long ln = i / chunks_per_row;
    const int kc = (int)(i - ln * chunks_per_row);
    const long long n = row0 + ln;
    long long v;
    if (map == MAP_ROPE) {
      const int half = hd >> 1;
      const long long head = n / hd;
      const int j = (int)(n - head * hd);
      const int b = j / half, jj = j - b * half;
      v = vbase + head * hd + (jj >> 3) * 16 + b * 8 + (jj & 7);
    } else if (map == MAP_GATE) {
      v = (n >> 3) * 16 + (n & 7);
    } else if (map == MAP_UP) {
      v = (n >> 3) * 16 + 8 + (n & 7);
    } else {
      v = vbase + n;
    }
    const long long nb = v >> 4;
    const int r = (int)(v & 15);
    const int kt = kc >> 2, g = kc & 3;
    T* d = dst + (((size_t)nb * KT + kt) * 64 + g * 16 + r) * KPL;
    const T* s = src + (size_t)ln * cols + (size_t)kc * KPL;
#pragma unroll
    for (int e = 0; e < KPL; ++e) d[e] = ((long long)kc * KPL + e < cols) ? s[e] : (T)0;
  }
}

__global__ void pad_gain_k(const float* src, int K, float* dst, int Kpad) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < Kpad) dst[k] = k < K ? src[k] : 0.f;
}

// Pure streaming read with the GEMV access pattern (non-temporal 1 KiB loads per wave, each wave
// a contiguous span, 8 loads in flight): the achievable-bandwidth ceiling of the weight stream.
__global__ void __launch_bounds__(512) stream_read_k(const uint4* base, long long n_tiles, float* sink) {
  const int lane = threadIdx.x & 63;
  const long long wave = ((long long)blockIdx.x * 512 + threadIdx.x) >> 6;
  const long long n_waves = ((long long)gridDim.x * 512) >> 6;
  const long long per = (n_tiles + n_waves - 1) / n_waves;
  const long long t0 = wave * per, t1 = t0 + per < n_tiles ? t0 + per : n_tiles;
  uint32_t acc = 0;
  long long t = t0;
  for (; t + 8 <= t1; t += 8) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ld_stream(base + (t + u) * 64 + lane);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; t < t1; ++t) {
    const uint4 v = ld_stream(base + t * 64 + lane);
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (acc == 0x9E3779B9u) sink[0] = 1.f;  // practically never; keeps the loads alive
}

// Plain copy of n 16-byte pieces (reads n*16 bytes, writes n*16 bytes): the known-size kernel
// against which the profiler's HBM byte counters are calibrated.
__global__ void __launch_bounds__(256) stream_copy_k(const uint4* __restrict__ src, uint4* __restrict__ dst, long long n) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) dst[i] = src[i];
}

// The one-row GEMV with parts of it switched off, for measurement only (results are not used): where a
// launch spends its time beyond the weight stream.  PARTS bit 0: the input row and gain staged through
// LDS (with the sum of squares); bit 1: bf16 decode and fp32 FMA (with the staged row, or with constants
// when bit 0 is off); bit 2: cross-wave reduction, RMS scale, residual add and store.  PARTS = 0 leaves
// the tile loads in the GEMV's geometry and schedule (two groups of GU tiles per wave in flight).
template <int PARTS>
__global__ void __launch_bounds__(1024) gemv_parts_k(const uint4* __restrict__ W, const float* __restrict__ X,
                                                    const float* __restrict__ G, const float* __restrict__ R,
                                                    float* __restrict__ Y, int KT) {
  constexpr bool STG = PARTS & 1, CMP = PARTS & 2, RED = PARTS & 4;
  extern __shared__ __align__(16) float xs[];
  __shared__ float red[MAXW][16];
  __shared__ float ssr[MAXW];
  const int tid = threadIdx.x, nw = blockDim.x >> 6, wave = tid >> 6, lane = tid & 63, g = lane >> 4, nb = blockIdx.x;
  int kt_lo, kt_hi;
  wave_span(KT, nw, wave, GU, kt_lo, kt_hi);
  const int ngroups = (kt_hi - kt_lo) / GU;
  const uint4* wp = W + ((size_t)nb * KT + kt_lo) * 64 + lane;
  float acc = 0.f, ss = 0.f;
  const int Kp = KT * 32, stride = blockDim.x * 4;
  float4 xv[4], gv[4];
  auto stage_load = [&](int base) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = base + j * stride;
      xv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      gv[j] = make_float4(1.f, 1.f, 1.f, 1.f);
      if (kk < Kp) { xv[j] = *(const float4*)(X + kk); gv[j] = *(const float4*)(G + kk); }
    }
  };
  auto stage_store = [&](int base) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = base + j * stride;
      if (kk < Kp) {
        const float4 x = xv[j], gg = gv[j];
        ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
        *(float4*)(xs + kk) = make_float4(x.x * gg.x, x.y * gg.y, x.z * gg.z, x.w * gg.w);
      }
    }
  };
  if (STG) stage_load(tid * 4);
  uint4 ta[GU], tb[GU];
  if (ngroups > 0) {
#pragma unroll
    for (int u = 0; u < GU; ++u) ta[u] = ld_stream(wp + u * 64);
  }
  if (ngroups > 1) {
#pragma unroll
    for (int u = 0; u < GU; ++u) tb[u] = ld_stream(wp + (GU + u) * 64);
  }
  if (STG) {
    stage_store(tid * 4);
    for (int base = tid * 4 + 4 * stride; base < Kp; base += 4 * stride) { stage_load(base); stage_store(base); }
    __syncthreads();
  }
  auto tile = [&](const uint4& w, int kt) {
    if (CMP) {
      float wf[8];
      WDec<8>::dec(w, wf);
      float4 a = make_float4(1.f, 2.f, 3.f, 4.f), b = make_float4(.5f, .25f, .125f, 2.f);
      if (STG) { a = *(const float4*)(xs + kt * 32 + g * 8); b = *(const float4*)(xs + kt * 32 + g * 8 + 4); }
      acc += wf[0] * a.x; acc += wf[1] * a.y; acc += wf[2] * a.z; acc += wf[3] * a.w;
      acc += wf[4] * b.x; acc += wf[5] * b.y; acc += wf[6] * b.z; acc += wf[7] * b.w;
    } else {
      acc += __uint_as_float((w.x ^ w.y ^ w.z ^ w.w) & 0x3fffffffu);
    }
  };
  auto use = [&](const uint4* tl, int gi) {
#pragma unroll
    for (int u = 0; u < GU; ++u) tile(tl[u], kt_lo + gi * GU + u);
  };
  auto fill = [&](uint4* tl, int gi) {
    const uint4* wn = wp + (size_t)gi * GU * 64;
#pragma unroll
    for (int u = 0; u < GU; ++u) tl[u] = ld_stream(wn + u * 64);
  };
  int gi = 0;
  for (; gi + 4 <= ngroups; gi += 2) { use(ta, gi); fill(ta, gi + 2); use(tb, gi + 1); fill(tb, gi + 3); }
  const int left = ngroups - gi;
  if (left == 3) { use(ta, gi); fill(ta, gi + 2); use(tb, gi + 1); use(ta, gi + 2); }
  else if (left == 2) { use(ta, gi); use(tb, gi + 1); }
  else if (left == 1) { use(ta, gi); }
  for (int kt = kt_lo + ngroups * GU; kt < kt_hi; ++kt) tile(ld_stream(wp + (size_t)(kt - kt_lo) * 64), kt);
  if (!RED) {
    if (acc == 123.456f || ss == 77.f) Y[nb * 16 + (lane & 15)] = acc;   // practically never; keeps the work alive
    return;
  }
  acc += __shfl_xor(acc, 16);
  acc += __shfl_xor(acc, 32);
  for (int o = 1; o < 64; o <<= 1) ss += __shfl_xor(ss, o);
  if (lane < 16) red[wave][lane] = acc;
  if (lane == 0) ssr[wave] = ss;
  __syncthreads();
  if (tid < 16) {
    float s = 0.f, q = 0.f;
    for (int w = 0; w < nw; ++w) s += red[w][tid];
    for (int w = 0; w < nw; ++w) q += ssr[w];
    s *= 1.0f / sqrtf(q / (float)(KT * 32) + 1e-5f);
    Y[nb * 16 + tid] = s + R[nb * 16 + tid];
  }
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
template <int KPL, int M, int EPI, bool ATT = false>
static hipError_t launch_valu_e(const GemmP& p, int waves, hipStream_t s) {
  while (waves > ValuWaves<M>::max) waves >>= 1;
  dim3 grid(p.NB), block(64 * waves);
  const size_t lds = M == 1 ? (size_t)p.KT * 4 * KPL * sizeof(float) : 0;
  if (lds > 48 * 1024) {  // beyond the default dynamic LDS limit: raise it for this kernel (once is enough)
    static size_t raised = 0;
    if (lds > raised) {
      hipError_t e = hipFuncSetAttribute((const void*)gemm_valu_k<KPL, M, EPI, ATT>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      raised = lds;
    }
  }
  if (p.ev_start && p.ev_stop)
    hipExtLaunchKernelGGL((gemm_valu_k<KPL, M, EPI, ATT>), grid, block, (uint32_t)lds, s, p.ev_start, p.ev_stop, 0, p);
  else
    hipLaunchKernelGGL((gemm_valu_k<KPL, M, EPI, ATT>), grid, block, lds, s, p);
  return hipGetLastError();
}

// The several-row-blocks-per-work-group form: bf16, one row, KT = 128, 160 or 256, at least one row block per
// work-group of a grid of ROWS_GRID; p.rows_form == 1 keeps the other kernel.
constexpr int ROWS_GRID = 256;   // one work-group per compute unit of the MI355X
template <int NG, int EPI, int GUX = GU>
static hipError_t launch_rows_e(const GemmP& p, hipStream_t s) {
  const size_t lds = (size_t)p.KT * 32 * sizeof(float);
  static size_t raised = 0;
  if (lds > 48 * 1024 && lds > raised) {
    hipError_t e = hipFuncSetAttribute((const void*)gemv_rows_k<NG, EPI, GUX>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    raised = lds;
  }
  const dim3 grid(p.NB < ROWS_GRID ? p.NB : ROWS_GRID), block(64 * ROWS_WAVES);
  if (p.ev_start && p.ev_stop)
    hipExtLaunchKernelGGL((gemv_rows_k<NG, EPI, GUX>), grid, block, (uint32_t)lds, s, p.ev_start, p.ev_stop, 0, p);
  else
    hipLaunchKernelGGL((gemv_rows_k<NG, EPI, GUX>), grid, block, lds, s, p);
  return hipGetLastError();
}
template <int NG, int GUX = GU>
static hipError_t launch_rows(const GemmP& p, int epi, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return launch_rows_e<NG, EPI_STORE, GUX>(p, s);
    case EPI_RESID: return launch_rows_e<NG, EPI_RESID, GUX>(p, s);
    case EPI_QKV: return launch_rows_e<NG, EPI_QKV, GUX>(p, s);
    case EPI_SWIGLU: return launch_rows_e<NG, EPI_SWIGLU, GUX>(p, s);
    case EPI_ARGMAX: return launch_rows_e<NG, EPI_ARGMAX, GUX>(p, s);
    default: return hipErrorInvalidValue;
  }
}

template <int KPL, int M>
static hipError_t launch_valu_m(const GemmP& p, int epi, int waves, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return launch_valu_e<KPL, M, EPI_STORE>(p, waves, s);
    case EPI_RESID:
      if constexpr (M == 1)
        if (p.att_S > 0) return launch_valu_e<KPL, 1, EPI_RESID, true>(p, waves, s);
      return launch_valu_e<KPL, M, EPI_RESID>(p, waves, s);
    case EPI_QKV: return launch_valu_e<KPL, M, EPI_QKV>(p, waves, s);
    case EPI_SWIGLU: return launch_valu_e<KPL, M, EPI_SWIGLU>(p, waves, s);
    case EPI_ARGMAX: return launch_valu_e<KPL, M, EPI_ARGMAX>(p, waves, s);
    default: return hipErrorInvalidValue;
  }
}

template <int KPL>
static hipError_t launch_valu_k(const GemmP& p, int epi, int waves, hipStream_t s) {
  if (p.M == 1) return launch_valu_m<KPL, 1>(p, epi, waves, s);
  if (p.M == 2) return launch_valu_m<KPL, 2>(p, epi, waves, s);
  // four and eight rows with 32-bit weights only: with 16-bit weights (twice the values per tile) they do not fit
  // a lane's registers
  if constexpr (KPL == 4) {
    if (p.M == 4) return launch_valu_m<KPL, 4>(p, epi, waves, s);
    if (p.M == 8) return launch_valu_m<KPL, 8>(p, epi, waves, s);
  }
  return hipErrorInvalidValue;
}

// (256 k tiles: up to six row blocks per work-group.  One row block per work-group / gemv_rows_k, us: 512 row blocks
// 30.8 / 28.0, 640 32.1 / 31.0, 2000 82.2 / 84.6, 3584 141.4 / 144.5: with many row blocks the start-up that gemv_rows_k
// saves no longer counts, and two work-groups per CU keep more requests out.)
bool gemv_rows_applies(const GemmP& p) {
  return p.wdtype == 1 && p.M == 1 && p.rows_form != 1 && p.NB >= ROWS_GRID && !p.XsOut &&
         (p.KT == 128 || p.KT == 160 || (p.KT == 256 && p.NB <= 6 * ROWS_GRID));
}
bool gemm_mfma_rows_applies(const GemmP& p, int epi, int col_blocks) {
  // (not with the residual epilogue and separate high and low parts: that instantiation does not fit 128 registers)
  const bool pack = p.M <= 8;
  return col_blocks == 1 && p.NB >= ROWS_GRID && p.rows_form != 1 &&
         (pack ? p.KT == 128 || p.KT == 160 : p.KT == 128 && epi != EPI_RESID);
}

hipError_t launch_gemm_valu(const GemmP& p, int epi, int waves, hipStream_t s) {
  if (waves < 1 || waves > MAXW || p.NB <= 0 || p.KT <= 0) return hipErrorInvalidValue;
  // attention partials as the input row: the output projection (no gain), at most ATT_SMAX splits, whole float4 groups of
  // features inside a head
  if (p.att_S > 0 && (epi != EPI_RESID || p.gain || p.att_S > ATT_SMAX || p.att_S > p.att_stride || p.K < 4 || p.att_hd % 4 ||
                      p.K % p.att_hd || !p.att_PM || !p.att_PL || !p.att_PA))
    return hipErrorInvalidValue;
  if (gemv_rows_applies(p))
    return p.KT == 128 ? launch_rows<2>(p, epi, s) : p.KT == 160 ? launch_rows<2, 5>(p, epi, s) : launch_rows<4>(p, epi, s);
  return p.wdtype == 1 ? launch_valu_k<8>(p, epi, waves, s) : launch_valu_k<4>(p, epi, waves, s);
}

template <int EPI>
static hipError_t launch_mfma_e(const GemmP& p, int waves, int col_blocks, hipStream_t s) {
  const dim3 grid(p.NB, col_blocks), block(64 * waves), rgrid(ROWS_GRID), rblock(64 * ROWS_WAVES);
  const bool pack = p.M <= 8;
#define MFMA_GO(K, GR, BL) hipExtLaunchKernelGGL(K, GR, BL, 0, s, p.ev_start, p.ev_stop, 0, p)
  if (gemm_mfma_rows_applies(p, EPI, col_blocks)) {
    // several row blocks per work-group, the activation tiles held in registers
    if (pack && p.KT == 128) MFMA_GO((gemm_mfma_rows_k<EPI, true, 8, 4>), rgrid, rblock);
    else if (pack) MFMA_GO((gemm_mfma_rows_k<EPI, true, 10, 5>), rgrid, rblock);
    else if constexpr (EPI != EPI_RESID) MFMA_GO((gemm_mfma_rows_k<EPI, false, 8, 2>), rgrid, rblock);
  } else if (pack) {
    MFMA_GO((gemm_mfma_k<EPI, true>), grid, block);
  } else {
    MFMA_GO((gemm_mfma_k<EPI, false>), grid, block);
  }
#undef MFMA_GO
  return hipGetLastError();
}

hipError_t launch_gemm_mfma(const GemmP& p, int epi, int waves, int col_blocks, hipStream_t s) {
  if (waves < 1 || waves > MAXW || p.NB <= 0 || p.KT <= 0 || p.wdtype != 1 || col_blocks < 1 ||
      p.M > col_blocks * 16 || p.M <= (col_blocks - 1) * 16)
    return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return launch_mfma_e<EPI_STORE>(p, waves, col_blocks, s);
    case EPI_RESID: return launch_mfma_e<EPI_RESID>(p, waves, col_blocks, s);
    case EPI_QKV: return launch_mfma_e<EPI_QKV>(p, waves, col_blocks, s);
    case EPI_SWIGLU: return launch_mfma_e<EPI_SWIGLU>(p, waves, col_blocks, s);
    case EPI_ARGMAX: return launch_mfma_e<EPI_ARGMAX>(p, waves, col_blocks, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_prep_split(const float* src, int rows, int rows_per_group, int64_t group_stride, int ld, int K,
                             int KT, const float* gain, int rms, float eps, uint16_t* Xs, float* rowscale,
                             hipStream_t s) {
  if (rows <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(prep_split_k, dim3(rows), dim3(256), 0, s, src, rows_per_group, (long long)group_stride, ld, K,
                     KT, gain, rms, eps, Xs, rowscale);
  return hipGetLastError();
}

static size_t attn_lds_bytes(int hd, int esize, int ct, int qb) {
  const int wpr = hd * esize / 4;
  return (size_t)2 * ct * (wpr + 1) * 4 + (size_t)qb * hd * 4 + (size_t)qb * ct * 4;
}

// Decode path (m == 1) for the shapes the register kernel is built for; S = number of splits.
// Returns hipErrorNotSupported for other shapes (the caller falls back to the staged kernels).
hipError_t launch_attention_decode(const AttnP& p, int S, hipStream_t s, int rows_per_wg) {
  if (p.m < 1 || S < 1 || S > p.nch_max) return hipErrorInvalidValue;
  const int G = p.n_q / p.n_kv;
  const bool many = rows_per_wg > 1;
  // one work-group per (split, kv head, group of token rows); G * rows per group <= 8 queries
#define DEL_ATT(KVT, HD, GG, RW)                                                                    \
  hipLaunchKernelGGL((attn_decode_k<KVT, HD, GG, RW>), dim3(S, p.n_kv, (p.m + RW - 1) / RW), dim3(RW > 1 ? 256 : 512), 0, s, p)
  if (p.kvdtype == 1 && p.hd == 128 && G == 1) { if (many) DEL_ATT(uint16_t, 128, 1, 8); else DEL_ATT(uint16_t, 128, 1, 1); }
  else if (p.kvdtype == 1 && p.hd == 64 && G == 4) { if (many) DEL_ATT(uint16_t, 64, 4, 2); else DEL_ATT(uint16_t, 64, 4, 1); }
  else if (p.kvdtype == 1 && p.hd == 128 && G == 8) DEL_ATT(uint16_t, 128, 8, 1);
  else if (p.kvdtype == 0 && p.hd == 64 && G == 1) { if (many) DEL_ATT(float, 64, 1, 4); else DEL_ATT(float, 64, 1, 1); }
  else return hipErrorNotSupported;
#undef DEL_ATT
  return hipGetLastError();
}

bool attention_decode_supported(int kvdtype, int hd, int G) {
  return (kvdtype == 1 && hd == 128 && (G == 1 || G == 8)) || (kvdtype == 1 && hd == 64 && G == 4) ||
         (kvdtype == 0 && hd == 64 && G == 1);
}

// Few token rows (m <= 16) on the matrix cores, S context splits of at least rps_min rows (a multiple of 32)
// each: writes S partials per (row, head); the caller merges them with launch_attention_merge (nsplit = S).
hipError_t launch_attention_flash_split(const AttnP& p, int S, int rps_min, hipStream_t s) {
  if (p.m < 1 || p.m > 16 || p.kvdtype != 1 || !p.VcT || p.TcapT % 32 != 0 || p.TcapT < p.Tcap || p.n_q % p.n_kv != 0 ||
      (p.hd != 64 && p.hd != 128) || S < 1 || S > p.nch_max || rps_min < 32 || rps_min % 32 != 0)
    return hipErrorInvalidValue;
  dim3 grid((S + 3) / 4, p.n_q), block(256);
  if (p.hd == 128) hipLaunchKernelGGL((attn_flash_split_k<128>), grid, block, 0, s, p, S, rps_min);
  else hipLaunchKernelGGL((attn_flash_split_k<64>), grid, block, 0, s, p, S, rps_min);
  return hipGetLastError();
}

// Merge p.nsplit partials per row (written by the decode kernel) into O (and XsOut).
hipError_t launch_attention_merge(const AttnP& p, hipStream_t s) {
  if (p.nsplit < 1 || p.nsplit > p.nch_max || p.hd > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_combine_k, dim3(p.m * p.n_q), dim3(128), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_attention(const AttnP& p, hipStream_t s) {
  const int es = p.kvdtype == 1 ? 2 : 4;
  // the staging registers hold ct rows of at most 4 x 256 threads x 16 bytes per matrix
  if (p.hd > 128 || p.hd % 16 != 0 || p.m < 1 || p.n_q % p.n_kv != 0 || p.ct < 16 || p.ct > 64 || p.ct % 16 != 0 ||
      p.ct * p.hd * es > 4 * 256 * 16)
    return hipErrorInvalidValue;
  dim3 grid(p.nch_max, p.n_kv), block(256);
  AttnP q = p;
  const int QR = p.m * (p.n_q / p.n_kv);
  q.qb = QR >= QBMAX ? QBMAX : ((QR + 3) & ~3);   // few query rows: less LDS, more work-groups per CU
  if (p.kvdtype == 1)
    hipLaunchKernelGGL((attn_partial_k<uint16_t>), grid, block, attn_lds_bytes(p.hd, 2, p.ct, q.qb), s, q);
  else
    hipLaunchKernelGGL((attn_partial_k<float>), grid, block, attn_lds_bytes(p.hd, 4, p.ct, q.qb), s, q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(attn_combine_k, dim3(p.m * p.n_q), dim3(128), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_embed(const void* Et, int wdtype, int KT, int vocab, const int* ids, int m, float* out, int ld,
                        int d_model, hipStream_t s) {
  if (wdtype == 1)
    hipLaunchKernelGGL((embed_k<8>), dim3(m), dim3(256), 0, s, Et, KT, vocab, ids, out, ld, d_model);
  else
    hipLaunchKernelGGL((embed_k<4>), dim3(m), dim3(256), 0, s, Et, KT, vocab, ids, out, ld, d_model);
  return hipGetLastError();
}

hipError_t launch_argmax_finish(const float* pval, const int* pidx, const float* psum, int rows, int NB, int* out_ids,
                                float* out_conf, hipStream_t s, const void* Et, int wdtype, int KT_e, int vocab,
                                float* emb_out, int d_model, unsigned long long* note, unsigned seq) {
  if ((emb_out && (rows != 1 || !Et)) || (note && !(psum && out_conf))) return hipErrorInvalidValue;
  // 16 waves where one row has more partials than four waves ask for at once, or a long embedding row to fetch; four
  // otherwise (a launch of 16 waves and their longer reduction cost the 256 partials of a small vocabulary 1 us)
  const bool big = rows == 1 && (NB > 256 * AF_UN || d_model > 4096);
  hipLaunchKernelGGL(argmax_finish_k, dim3(rows), dim3(big ? 1024 : 256), 0, s, pval, pidx, psum, NB, out_ids, out_conf, Et,
                     wdtype == 1 ? 8 : 4, KT_e, vocab, emb_out, d_model, note, seq);
  return hipGetLastError();
}

hipError_t launch_accept(int* state, const int* draft_ids, int* shadow_ids, int L, int m, int E, int gamma,
                         int* result, hipStream_t s) {
  if (gamma > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(accept_k, dim3(1), dim3(64), 0, s, state, draft_ids, shadow_ids, L, m, E, gamma, result);
  return hipGetLastError();
}

hipError_t launch_set_state(int* state, int add_T, int set_T, const int* pending_src, int pending_val,
                            hipStream_t s) {
  hipLaunchKernelGGL(set_state_k, dim3(1), dim3(64), 0, s, state, add_T, set_T, pending_src, pending_val);
  return hipGetLastError();
}

hipError_t launch_tile_scatter(const void* src, int wdtype, int64_t row0, int64_t nrows, int64_t cols, int map,
                               int vbase, int hd, void* dst, int KT, hipStream_t s) {
  const int kpl = wdtype == 1 ? 8 : 4;
  const int64_t total = nrows * ((cols + kpl - 1) / kpl);
  if (total <= 0) return hipSuccess;
  const int64_t want = (total + 255) / 256;
  const int blocks = (int)(want < 65535 * 4 ? want : 65535 * 4);
  if (wdtype == 1)
    hipLaunchKernelGGL((tile_scatter_k<8, uint16_t>), dim3(blocks), dim3(256), 0, s, (const uint16_t*)src,
                       (long long)row0, (long long)nrows, (long long)cols, map, vbase, hd, (uint16_t*)dst, KT);
  else
    hipLaunchKernelGGL((tile_scatter_k<4, float>), dim3(blocks), dim3(256), 0, s, (const float*)src, (long long)row0,
                       (long long)nrows, (long long)cols, map, vbase, hd, (float*)dst, KT);
  return hipGetLastError();
}

hipError_t launch_pad_gain(const float* src, int K, float* dst, int Kpad, hipStream_t s) {
  hipLaunchKernelGGL(pad_gain_k, dim3((Kpad + 255) / 256), dim3(256), 0, s, src, K, dst, Kpad);
  return hipGetLastError();
}

hipError_t launch_stream_copy(const void* src, void* dst, int64_t bytes, hipStream_t s) {
  const long long n = bytes / 16;
  if (n <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stream_copy_k, dim3(256 * 16), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n);
  return hipGetLastError();
}

hipError_t launch_stream_read(const void* base, int64_t bytes, float* sink, hipStream_t s) {
  const long long n_tiles = bytes / 1024;
  if (n_tiles <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stream_read_k, dim3(256 * 8), dim3(512), 0, s, (const uint4*)base, n_tiles, sink);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Measurement kernel: issue rate of the two bf16 matrix instructions with NACC independent accumulators per
// wave and no memory traffic in the loop (one wave per SIMD, one work-group per compute unit).  SHAPE 0:
// v_mfma_f32_16x16x32_bf16 (the instruction the weight tiles are laid out for), 1: v_mfma_f32_32x32x16_bf16.
// The accumulators start from memory so that they are distinct values; results are discarded.
// ---------------------------------------------------------------------------------------
typedef float floatx16 __attribute__((ext_vector_type(16)));
template <int SHAPE, int NACC>
__global__ void __launch_bounds__(256) mfma_rate_k(const float* init, float* out, int iters) {
  const int lane = threadIdx.x & 63;
  bf16x8 a, b;
  {
    const uint4 ua = *(const uint4*)(init + 4 * lane), ub = *(const uint4*)(init + 256 + 4 * lane);
    a = __builtin_bit_cast(bf16x8, ua);
    b = __builtin_bit_cast(bf16x8, ub);
  }
  float s = 0.f;
  if (SHAPE == 0) {
    floatx4 acc[NACC];
#pragma unroll
    for (int n = 0; n < NACC; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[n][j] = init[512 + (n * 4 + j) * 64 + lane];
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int n = 0; n < NACC; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < NACC; ++n) s += acc[n][0] + acc[n][1] + acc[n][2] + acc[n][3];
  } else {
    floatx16 acc[NACC];
#pragma unroll
    for (int n = 0; n < NACC; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[n][j] = init[512 + (n * 16 + j) * 64 + lane];
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int n = 0; n < NACC; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < NACC; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) s += acc[n][j];
  }
  if (s == 12345.678f) out[threadIdx.x] = s;   // keeps the loop alive; the buffers hold zeros
}

// init: 512 + 64 * 64 floats (zeros will do), out: 256 floats
hipError_t launch_mfma_rate(int shape, int n_acc, const float* init, float* out, int iters, hipStream_t s) {
  const dim3 grid(256), block(256);
#define MFMA_RATE(S, N)                                                                     \
  if (shape == S && n_acc == N) {                                                           \
    hipLaunchKernelGGL((mfma_rate_k<S, N>), grid, block, 0, s, init, out, iters);           \
    return hipGetLastError();                                                               \
  }
  MFMA_RATE(0, 2) MFMA_RATE(0, 4) MFMA_RATE(0, 8) MFMA_RATE(0, 16)
  MFMA_RATE(1, 1) MFMA_RATE(1, 2) MFMA_RATE(1, 4)
#undef MFMA_RATE
  return hipErrorInvalidValue;
}

hipError_t launch_gemv_parts(const void* W, const float* X, const float* G, const float* R, float* Y, int NB, int KT,
                             int waves, int parts, hipStream_t s) {
  if (NB < 1 || KT < 1 || KT > 480 || (waves != 4 && waves != 8 && waves != 16) || parts < 0 || parts > 7)
    return hipErrorInvalidValue;
  const dim3 grid(NB), block(64 * waves);
  const size_t lds = (size_t)KT * 32 * sizeof(float);
  switch (parts) {
#define GP(v) case v: hipLaunchKernelGGL((gemv_parts_k<v>), grid, block, lds, s, (const uint4*)W, X, G, R, Y, KT); break;
    GP(0) GP(1) GP(2) GP(3) GP(4) GP(5) GP(6) GP(7)
#undef GP
  }
  return hipGetLastError();
}

}  // namespace del
