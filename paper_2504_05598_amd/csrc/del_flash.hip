// Attention on the matrix cores: causal over many token rows (prompt passes), and of one token row (draft steps).
#include "del_device.h"

#include <algorithm>

namespace del {

namespace {

// Largest of the four values that the lanes of one query hold (lanes l, l ^ 16, l ^ 32, l ^ 48); no LDS traffic.
__device__ __forceinline__ float max_of_query(float v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const unsigned a = __float_as_uint(v);
  const u32x2 s = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(a, a, false, false));
  const unsigned b = __float_as_uint(fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1])));
  const u32x2 t = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(b, b, false, false));
  return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}

// Eight values -> bf16 high parts and bf16 remainders (16 mantissa bits together), as matrix-core operands.
__device__ __forceinline__ void split8_op(const float* v, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    hi[e] = (__bf16)v[e];
    lo[e] = (__bf16)(v[e] - (float)hi[e]);
  }
}

}  // namespace

// One wave = 32 consecutive token rows (two blocks of 16) of one query head, four waves per work-group; all four read
// the same keys and values, staged in LDS 64 cache rows at a time by loads that write LDS directly, two stages.
// Per 32 cache rows and block of 16 token rows:
//   S^T[32 rows][16 queries] = K[32][hd] * Q^T      (A = cache rows as stored, B = queries as bf16 high + low parts)
//   online soft-max per query, in powers of two (the queries carry the factor log2 e)
//   O^T[hd][16 queries] += V^T[hd][32 rows] * P     (A = the feature-major copy of the values, B = the probabilities,
//                                                    high + low parts)
// The A operand of the first product takes cache row t + 8*(i/4) + i%4 (+4 for the second block of 16) as its row i, so
// that the 8 scores a lane ends up with are 8 consecutive cache rows: exactly the B operand slice it must supply to the
// second product.  What bounds it: per 32 rows a wave issues 64 matrix instructions (1024 clocks) and about 200 vector
// instructions for two soft-max blocks; one block per wave with keys and values from the cache (the form before) read
// 16 KiB through the vector cache for 32 instructions and ran at a seventh of the matrix rate.  Per launch: 7B shape,
// 1024 rows on an empty cache 97 -> 51 us; 13B shape, mean of four passes up to 4001 rows 481 -> 140 us.  The running maximum is
// only raised when it grows by more than a factor 2^8 (the sums stay far inside fp32's range), which leaves the
// rescaling of the output out of nearly every step.
// LDS layout: 16-byte chunks, the chunk index of a key row (feature row) XORed with bits of the row number such that the
// 16 lanes that read together hit 16 different bank groups; the loads fetch chunks in that order, whole rows at a time.
template <int HD>
__global__ void __launch_bounds__(256, 2) attn_flash_k(AttnP p) {
  constexpr int KT = HD / 32, DT = HD / 16, CH = HD / 8, TR = 64;
  constexpr int NL = TR * CH / 64 / 4;               // 1 KiB pieces of the keys (and of the values) per wave and stage
  __shared__ __align__(16) uint4 k0s[TR * CH], k1s[TR * CH], v0s[TR * CH], v1s[TR * CH];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4, qi = lane & 15;
  const int h = blockIdx.y, kvh = h / (p.n_q / p.n_kv);
  const int rb = ((int)gridDim.x - 1 - (int)blockIdx.x) * 128;   // the blocks with the longest context start first
  const int r0 = rb + wave * 32;
  const int T0 = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off;       // cache position of token row 0
  const int wg_end = T0 + min(rb + 128, p.m);        // cache rows the work-group needs: [0, wg_end)
  const int t_end = r0 < p.m ? T0 + min(r0 + 32, p.m) : 0;                     // ... and this wave
  const float scale = 1.44269504088896340736f / sqrtf((float)HD);
  bf16x8 qh[2][KT], ql[2][KT];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    // rows past the pass re-read its last row; their results are dropped
    const float* qp = p.Q + (size_t)min(r0 + b * 16 + qi, p.m - 1) * p.ldq + (size_t)h * HD + 8 * g;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const float4 x = *(const float4*)(qp + 32 * kt), y = *(const float4*)(qp + 32 * kt + 4);
      const float v[8] = {x.x * scale, x.y * scale, x.z * scale, x.w * scale,
                          y.x * scale, y.y * scale, y.z * scale, y.w * scale};
      split8_op(v, qh[b][kt], ql[b][kt]);
    }
  }
  floatx4 o[2][DT];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[b][dt] = (floatx4){0.f, 0.f, 0.f, 0.f};
  float mrun[2] = {-INFINITY, -INFINITY}, lrun[2] = {0.f, 0.f};   // lrun: this lane's rows only
  const uint16_t* Kb = (const uint16_t*)p.Kc + (size_t)kvh * p.Tcap * HD;
  const uint16_t* Vt = (const uint16_t*)p.VcT + (size_t)kvh * HD * p.TcapT;
  auto swz = [](int r) { return HD == 128 ? (r & 3) | ((r >> 3) & 3) << 2 : ((r >> 1) & 1) | ((r >> 3) & 3) << 1; };
  typedef const void __attribute__((address_space(1)))* gptr_t;
  typedef void __attribute__((address_space(3)))* lptr_t;
  auto request = [&](int t0, uint4* ks, uint4* vs) {
#pragma unroll
    for (int n = 0; n < NL; ++n) {
      const int s = (wave * NL + n) * 64 + lane, r = s / CH, c = (s % CH) ^ swz(r);
      // rows past the last one the work-group needs are read from that row and masked in the scores
      __builtin_amdgcn_global_load_lds((gptr_t)(Kb + (size_t)min(t0 + r, wg_end - 1) * HD + c * 8),
                                       (lptr_t)(ks + (wave * NL + n) * 64), 16, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < NL; ++n) {
      const int s = (wave * NL + n) * 64 + lane, f = s >> 3, c = (s & 7) ^ ((f >> 1) & 7);
      // (the feature rows are padded to whole 32s: the last 64 may reach past them)
      __builtin_amdgcn_global_load_lds((gptr_t)(Vt + (size_t)f * p.TcapT + min(t0 + c * 8, p.TcapT - 8)),
                                       (lptr_t)(vs + (wave * NL + n) * 64), 16, 0, 0);
    }
  };
  const int rho = 8 * (qi >> 2) + (qi & 3);
  auto compute = [&](int t, int sub, const uint4* ks, const uint4* vs) __attribute__((always_inline)) {
    const int ra = sub * 32 + rho, rbb = ra + 4;
    floatx4 s[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b) s[b][0] = s[b][1] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const bf16x8 x0 = __builtin_bit_cast(bf16x8, ks[ra * CH + ((kt * 4 + g) ^ swz(ra))]);
      const bf16x8 x1 = __builtin_bit_cast(bf16x8, ks[rbb * CH + ((kt * 4 + g) ^ swz(rbb))]);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        s[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, qh[b][kt], s[b][0], 0, 0, 0);
        s[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, qh[b][kt], s[b][1], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        s[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, ql[b][kt], s[b][0], 0, 0, 0);
        s[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, ql[b][kt], s[b][1], 0, 0, 0);
      }
    }
    bf16x8 ph[2], pl[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      // this lane: scores of cache rows t + 8g + e, e = 0..7, for its query
      float sv[8] = {s[b][0][0], s[b][0][1], s[b][0][2], s[b][0][3], s[b][1][0], s[b][1][1], s[b][1][2], s[b][1][3]};
      if (t + 31 > T0 + r0 + b * 16) {               // uniform: some query of the block does not see all 32 rows
        const int pos = T0 + r0 + b * 16 + qi;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (t + 8 * g + e > pos) sv[e] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
      mx = max_of_query(mx);
      const bool grow = mx > mrun[b] + 8.0f;         // always on the first tile: row 0 is never masked
      if (__builtin_amdgcn_ballot_w64(grow)) {
        const float c = grow ? __builtin_amdgcn_exp2f(mrun[b] - mx) : 1.0f;
        if (grow) mrun[b] = mx;
        lrun[b] *= c;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int j = 0; j < 4; ++j) o[b][dt][j] *= c;
      }
      float pv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(sv[e] - mrun[b]);
      lrun[b] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
      split8_op(pv, ph[b], pl[b]);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int f = dt * 16 + qi;
      const bf16x8 x = __builtin_bit_cast(bf16x8, vs[f * 8 + ((sub * 4 + g) ^ ((f >> 1) & 7))]);
#pragma unroll
      for (int b = 0; b < 2; ++b) o[b][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, ph[b], o[b][dt], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < 2; ++b) o[b][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pl[b], o[b][dt], 0, 0, 0);
    }
  };
  // one stage: it has arrived for every wave once all have passed the barrier, which also says that the other one is no
  // longer being read.  A wave whose rows end earlier only takes part in the loads and barriers.
  auto step = [&](int t0, const uint4* ks, const uint4* vs, uint4* kn, uint4* vn) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (t0 + TR < wg_end) request(t0 + TR, kn, vn);
    __builtin_amdgcn_sched_barrier(0);
    if (t0 < t_end) compute(t0, 0, ks, vs);
    if (t0 + 32 < t_end) compute(t0 + 32, 1, ks, vs);
  };
  request(0, k0s, v0s);
  for (int t0 = 0; t0 < wg_end; t0 += 2 * TR) {
    step(t0, k0s, v0s, k1s, v1s);
    if (t0 + TR < wg_end) step(t0 + TR, k1s, v1s, k0s, v0s);
  }
  // this lane: features 16*dt + 4g + j of head h for its token rows, as split tiles (the output projection's input)
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    float l = lrun[b];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const int row = r0 + b * 16 + qi;
    if (row >= p.m) continue;
    const float inv = 1.0f / l;
    uint16_t* xs = p.XsOut + (size_t)(row >> 4) * p.xs_cb_stride;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const float v[4] = {o[b][dt][0] * inv, o[b][dt][1] * inv, o[b][dt][2] * inv, o[b][dt][3] * inv};
      const int k = h * HD + 16 * dt + 4 * g;       // first of 4 consecutive features
      uint2 hi, lo;
      split4(v, hi, lo);
      uint16_t* dst = xs + (size_t)(k >> 5) * 1024 + (((k & 31) >> 3) * 16 + (row & 15)) * 8 + (k & 7);
      *(uint2*)dst = hi;
      *(uint2*)(dst + 512) = lo;
    }
  }
}

// Attention of one token row: one work-group per (split of the context, kv head), NWV waves, a wave = 32 cache rows at a
// time for all query heads of the group at once (they are the columns of the matrix-core products above; columns past
// the group repeat its first head and are dropped).  Bound by latency: position -> cache rows -> two short products ->
// merge of the waves through LDS.  The vector form before it (one lane group per cache row, every query head on its own:
// a dot product, three shuffles and two exponentials per head and row, the same again to merge the lane groups) grew with
// the heads of a group.  Per launch, us: eight heads per kv head 21.1 -> 7.2 (70B shape, 1050 rows), four 9.8 -> 4.9 (1B shape);
// with one head per kv head the vector kernel stays (7B shape 8.1 + 9.7 with the output projection against 7.4 + 10.5, 13B
// 11.4 against 14.5).
template <int HD, int NWV>
__global__ void __launch_bounds__(64 * NWV) attn_row_k(AttnP p) {
  constexpr int KT = HD / 32, DT = HD / 16, GMAX = 16;
  __shared__ float sm[NWV][GMAX], sl[NWV][GMAX];
  __shared__ __align__(16) float so[NWV][GMAX][HD + 4];   // (+ 4: the 16 columns of a store fall into different banks)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, qi = lane & 15;
  const int split = blockIdx.x, kvh = blockIdx.y, S = gridDim.x, G = p.n_q / p.n_kv;
  const float* qp = p.Q + (size_t)(kvh * G + (qi < G ? qi : 0)) * HD + 8 * g;
  float4 qa[KT], qb[KT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) { qa[kt] = *(const float4*)(qp + 32 * kt); qb[kt] = *(const float4*)(qp + 32 * kt + 4); }
  const int T_end = (p.ctx_len1 ? p.ctx_len1 - 1 : p.state[0]) + p.row_off + 1;   // the row attends cache rows [0, T_end)
  const int rps = ((T_end + S - 1) / S + 31) / 32 * 32;
  const int t_lo = split * rps, t_hi = min(T_end, t_lo + rps);
  const uint16_t* Kb = (const uint16_t*)p.Kc + (size_t)kvh * p.Tcap * HD + 8 * g;
  const uint16_t* Vt = (const uint16_t*)p.VcT + ((size_t)kvh * HD + qi) * p.TcapT + 8 * g;
  const int rho = 8 * (qi >> 2) + (qi & 3);
  float mrun = -INFINITY, lrun = 0.f;                  // lrun: this lane's cache rows only
  floatx4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = (floatx4){0.f, 0.f, 0.f, 0.f};
  bf16x8 qh[KT], ql[KT];
  auto load = [&](int t0, uint4* a0, uint4* a1, uint4* av) {
    // rows past the last one are read from it and masked in the scores
    const uint16_t* k0 = Kb + (size_t)min(t0 + rho, T_end - 1) * HD;
    const uint16_t* k1 = Kb + (size_t)min(t0 + rho + 4, T_end - 1) * HD;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      a0[kt] = *(const uint4*)(k0 + 32 * kt);
      a1[kt] = *(const uint4*)(k1 + 32 * kt);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) av[dt] = *(const uint4*)(Vt + (size_t)(16 * dt) * p.TcapT + t0);
  };
  auto compute = [&](int t0, const uint4* a0, const uint4* a1, const uint4* av) __attribute__((always_inline)) {
    floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const bf16x8 x0 = __builtin_bit_cast(bf16x8, a0[kt]), x1 = __builtin_bit_cast(bf16x8, a1[kt]);
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, qh[kt], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, qh[kt], s1, 0, 0, 0);
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0, ql[kt], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1, ql[kt], s1, 0, 0, 0);
    }
    float sv[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (t0 + 8 * g + e >= t_hi) sv[e] = -INFINITY;   // (row t0 itself is always inside)
      mx = fmaxf(mx, sv[e]);
    }
    mx = fmaxf(mrun, max_of_query(mx));
    const float c = expf(mrun - mx);                   // first tile: exp(-inf) = 0
    mrun = mx;
    float pv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pv[e] = expf(sv[e] - mx);
    lrun = lrun * c + (((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7])));
    bf16x8 ph, pl;
    split8_op(pv, ph, pl);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int j = 0; j < 4; ++j) o[dt][j] *= c;
      const bf16x8 x = __builtin_bit_cast(bf16x8, av[dt]);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, ph, o[dt], 0, 0, 0);
      o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pl, o[dt], 0, 0, 0);
    }
  };
  constexpr int STEP = 32 * NWV;
  const int first = t_lo + wave * 32;
  if (first < t_hi) {                                  // wave-uniform
    // two register sets used in turn, the next tile's rows requested before the current tile is multiplied
    uint4 ka0[KT], ka1[KT], va[DT], kb0[KT], kb1[KT], vb[DT];
    load(first, ka0, ka1, va);
    const float scale = 1.0f / sqrtf((float)HD);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const float v[8] = {qa[kt].x * scale, qa[kt].y * scale, qa[kt].z * scale, qa[kt].w * scale,
                          qb[kt].x * scale, qb[kt].y * scale, qb[kt].z * scale, qb[kt].w * scale};
      split8_op(v, qh[kt], ql[kt]);
    }
    for (int t0 = first; t0 < t_hi; t0 += 2 * STEP) {
      if (t0 + STEP < t_hi) load(t0 + STEP, kb0, kb1, vb);
      compute(t0, ka0, ka1, va);
      if (t0 + STEP >= t_hi) break;
      if (t0 + 2 * STEP < t_hi) load(t0 + 2 * STEP, ka0, ka1, va);
      compute(t0 + STEP, kb0, kb1, vb);
    }
  }
  lrun += __shfl_xor(lrun, 16);
  lrun += __shfl_xor(lrun, 32);
  if (qi < G) {
    if (g == 0) { sm[wave][qi] = mrun; sl[wave][qi] = lrun; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *(floatx4*)&so[wave][qi][16 * dt + 4 * g] = o[dt];
  }
  __syncthreads();
  // the waves in a fixed order; one partial per (query head, split), or the result itself
  for (int i = tid; i < G * HD; i += 64 * NWV) {
    const int c = i / HD, d = i - c * HD;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NWV; ++w) M = fmaxf(M, sm[w][c]);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      const float f = sm[w][c] > -INFINITY ? expf(sm[w][c] - M) : 0.f;
      L += f * sl[w][c];
      A += f * so[w][c][d];
    }
    const int h = kvh * G + c;
    if (S == 1 && p.nsplit < 0) {
      p.O[(size_t)h * HD + d] = A / L;
      continue;
    }
    const size_t prow = (size_t)h * p.nch_max + split;
    if (d == 0) { p.PM[prow] = M; p.PL[prow] = L; }
    p.PA[prow * HD + d] = A;
  }
}

// Work-groups along the context for a row that attends n cache rows: one tile of 32 rows per wave of four waves, as many
// partials as the output projection's staging merges at most.
int attention_row_splits(int n) { return std::min(8, (n + 127) / 128); }

// Groups of several query heads: one launch, vector form -> this one, 64 heads on 8 kv heads of width 128 at 1050 rows
// 21.1 -> 7.2 us, 32 on 8 of width 64 at 540 rows 9.8 -> 4.9, 8 on 2 of width 64 at 70 rows 8.5 -> 3.7.  With a kv head per
// query head 15 of 16 columns are idle and the values come in 64-byte pieces; there the vector form stays: 32 heads at
// 1050 rows 8.1 us and 9.7 for the projection that merges its four partials, here 7.4 and 10.5 (eight partials); 40
// heads at 2000 rows 11.4 against 14.5.
bool attention_row_supported(int kvdtype, int hd, int G) {
  return kvdtype == 1 && (hd == 64 || hd == 128) && G > 1 && G <= 16;
}

// p.m == 1.  S context splits; S == 1 with p.nsplit < 0 writes the output row, otherwise the partials.  Eight waves where
// four would each see more than one tile of the longest context the splits may have.
hipError_t launch_attention_row(const AttnP& p, int S, int n_max, hipStream_t s) {
  if (p.m != 1 || !attention_row_supported(p.kvdtype, p.hd, p.n_q / p.n_kv) || !p.VcT || p.TcapT % 32 != 0 ||
      p.TcapT < p.Tcap || p.n_q % p.n_kv != 0 || S < 1 || S > p.nch_max || (p.nsplit >= 0 && (!p.PM || !p.PL || !p.PA)))
    return hipErrorInvalidValue;
  const dim3 grid(S, p.n_kv);
  const bool eight = (n_max + S - 1) / S > 128;
  if (p.hd == 128) {
    if (eight) hipLaunchKernelGGL((attn_row_k<128, 8>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((attn_row_k<128, 4>), grid, dim3(256), 0, s, p);
  } else {
    if (eight) hipLaunchKernelGGL((attn_row_k<64, 8>), grid, dim3(512), 0, s, p);
    else hipLaunchKernelGGL((attn_row_k<64, 4>), grid, dim3(256), 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_attention_flash(const AttnP& p, hipStream_t s) {
  if (p.m < 1 || p.kvdtype != 1 || !p.VcT || p.TcapT % 32 != 0 || p.TcapT < p.Tcap || p.n_q % p.n_kv != 0 || !p.XsOut ||
      (p.hd != 64 && p.hd != 128))
    return hipErrorInvalidValue;
  dim3 grid((p.m + 127) / 128, p.n_q), block(256);
  if (p.hd == 128) hipLaunchKernelGGL((attn_flash_k<128>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((attn_flash_k<64>), grid, block, 0, s, p);
  return hipGetLastError();
}

}  // namespace del
