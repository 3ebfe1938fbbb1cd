// Scores of many queries against a cache (im_index_score with more queries than score_short takes; Section
// 3.1, Eq. (5)): imp[key] = max over the queries that may see the key of S = sum_j alpha_j ReLU(q_j . k), in fp64.
//
// The fp64 value is needed for ONE query per key, the maximal one.  So the scores of all (query, key) pairs are
// taken on the fp16 matrix cores, at 32 times the fp64 rate, together with a rigorous bound of their error, and only
// pairs whose upper bound reaches the best lower bound of their key are evaluated in fp64 (about 1.03 per
// key on the benchmark's inputs).  The result is the same fp32 number an fp64 pass over all pairs gives.
//   k_score_features : QK-Norm, head gates, fp16 operands and error bounds, per block of 16 queries
//   k_score_scan     : upper bounds of all pairs; per key and lane group the largest, its query block, the second
//   k_score_exact    : fp64 scores of the candidates; keys with more candidates than the scan could name are listed
//   k_score_listed   : those keys against all queries: the bound again, fp64 where it still exceeds the score
//
// Upper bound.  With ReLU(z) = (z + |z|) / 2:  S = c . k + sum_j (alpha_j / 2) |q_j . k|,  c = sum_j (alpha_j / 2) q_j:
// one more matrix product, but a single FMA (with a free |.|) per pair and head on the vector ALU.
// q_j, c and k are scaled by powers of two so that their norms lie in [2^11, 2^12) (scaled norms below: N_j, N_c) and
// rounded to fp16; values below 2^-14, fp16's smallest normal, become 0.  With the residuals r of the rounding (known
// exactly), the scaled |alpha_j| / 2 as a_j, the inverse scale of c as t, and ||k|| < 2^12:
//   |error| <= 2^12 [ t ||r_c|| + sum_j a_j ||r_j|| + 2^-16 (t N_c + sum_j a_j N_j) ]            (Cauchy-Schwarz)
// where the 2^-16 covers the fp32 sums inside the products (64 terms of at most 2^-23 each: 2^-17), the key's values
// lost below 2^-14 (2^-22) and the at most 17 FMAs of the gated sum (2^-19).
#pragma once
#include "im_kernels.h"

#define IM_SCORE_GROUPS 8   // most query groups of a scan over a short cache

typedef _Float16 im_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 im_h4 __attribute__((ext_vector_type(4)));
typedef float im_f4 __attribute__((ext_vector_type(4)));

// Block of 16 queries, HM (8 or 16) indexer heads at most.  fp16 operands first: head j (index H_idx: the vector c)
// takes 16 DI values in the order in which lane (row l16 = query, kq) of the product reads them; then rows of 16
// floats: a_j per head, t, the error bound, and the query positions (int).
template <int DI, int HM>
struct ScoreBlock {
  static constexpr int HEAD = 16 * DI * 2;                          // bytes of one head
  static constexpr int OFF = (HM + 1) * HEAD;                       // the rows of floats
  static constexpr int T = HM, ERR = HM + 1, POS = HM + 2, ROWS = HM + 3;
  static constexpr int BYTES = (OFF + ROWS * 64 + 1023) / 1024 * 1024;   // whole 1 KB wave copies
};

// power of two that brings a norm into [2^11, 2^12); 1 for a zero or non-finite one
__device__ __forceinline__ float score_scale(float norm) {
  const int e = (int)((__float_as_uint(norm) >> 23) & 255u) - 127;
  return (norm > 0.f && e > -100 && e < 100) ? __uint_as_float((uint32_t)(127 + 11 - e) << 23) : 1.f;
}
__device__ __forceinline__ bool score_sane(float x) {   // zero, or of a size whose scaled forms stay normal numbers
  const float m = fabsf(x);
  return m == 0.f || (m > 8.6e-19f && m < 1.2e18f);     // 2^-60 .. 2^60
}
__device__ __forceinline__ _Float16 score_half(float x) {
  return (fabsf(x) < 6.103515625e-05f) ? (_Float16)0.f : (_Float16)x;
}

// grid (ceil(n_q / 16), B), 16 waves: one block of 16 queries, one per wave.
// qraw [B n_q, H_idx, DI], araw [B n_q, H_idx]: the raw projections (fp64).  qf: the normalised features (fp32, as
// the exact evaluation reads them), al16 [B n_q, 16]: alpha (fp32, zero past H_idx).
// Lane: dim lane % DI of head (pass * 64 / DI + lane / DI), all heads' loads first.  Per-head sums: at DI = 64 for all heads at
// once by a butterfly (head h of it: lane 15 of row rho of register i, 4 i + 2 (rho & 1) + (rho >> 1)), so that roots, scales
// and bounds are taken once per 4 heads; at DI = 16 inside the 16-lane rows.  The block's operands are put together
// in LDS and leave in one piece.  Bound: reads 8 and writes 6 bytes per feature; a short prompt's few workgroups: one
// chain of latencies (a wave with 4 queries and 8 heads in turn took 27 us for 562 queries, 192 us for 65536).
template <int DI, int HM>
__global__ __launch_bounds__(1024) void k_score_features(const double* __restrict__ qraw, const double* __restrict__ araw,
                                                         const int32_t* __restrict__ q_pos,
                                                         const bf16_t* __restrict__ norm_w, float rms_eps,
                                                         double alpha_denom, int n_q, int H_idx,
                                                         float* __restrict__ qf, float* __restrict__ al16,
                                                         char* __restrict__ blocks, int32_t* __restrict__ n_listed) {
  using SB = ScoreBlock<DI, HM>;
  constexpr int HP = 64 / DI, NP = HM / HP;   // heads per pass of a wave, passes
  __shared__ __attribute__((aligned(16))) char sb[SB::BYTES];
  const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.y, d = lane % DI, hl = lane / DI;
  const int m = __builtin_amdgcn_readfirstlane(tid >> 6), s = blockIdx.x * 16 + m;
  const size_t row = (size_t)b * n_q + min(s, n_q - 1);
  // all loads first (absent heads repeat the last, unused)
  double v[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) v[i] = qraw[(row * H_idx + min(i * HP + hl, H_idx - 1)) * DI + d];
  const double a_raw = araw[row * H_idx + min(lane & 15, H_idx - 1)];
  const float nw = norm_w ? bf2f(norm_w[d]) : 1.f;
  const int my_pos = q_pos[row];
  if (blockIdx.x == 0 && tid == 0) n_listed[b] = 0;
  for (int i = tid; i < SB::BYTES / 4; i += 1024) ((uint32_t*)sb)[i] = 0;
  __syncthreads();
  float* rows = (float*)(sb + SB::OFF);
  // place of dim d in a head's operand: lane (m, kq) holds dims DI/4 kq .. of query m, in steps of 8 (DI = 64)
  constexpr int DPL = DI / 4;
  const int kq = d / DPL, e = d % DPL;
  const int place = ((DI == 64) ? (e / 8) * 1024 + kq * 256 + (e % 8) * 2 : kq * 128 + e * 2) + m * (DI == 64 ? 16 : 8);
  if (s >= n_q) {
    if (lane == 0) { rows[SB::ERR * 16 + m] = -INFINITY; ((int*)rows)[SB::POS * 16 + m] = INT_MAX; }
  } else {
    const float al_l = (float)(a_raw / alpha_denom);   // of head lane % 16
    if (lane < 16) al16[row * 16 + lane] = (lane < H_idx) ? al_l : 0.f;
    double c = 0.0;                       // this lane's share of c[d]
    float err = 0.f;                      // sum of the heads' terms
    bool sane = true;
    float q[NP];
    if constexpr (DI == 64) {
      constexpr int NR = HM / 4;          // registers of the butterfly
      const int rho = lane >> 4;
      const bool holds = (lane & 15) == 15;
      double sq[HM], ss[NR];
#pragma unroll
      for (int j = 0; j < HM; ++j) sq[j] = v[j] * v[j];
      wave_sums_butterfly_d<HM>(sq, ss);
#pragma unroll
      for (int i = 0; i < NR; ++i) ss[i] = sqrt(ss[i] / (double)DI + (double)rms_eps);
      float t[HM], n2[NR], r2[NR], sc[NR];
#pragma unroll
      for (int j = 0; j < HM; ++j) {
        q[j] = (float)(v[j] / readlane_d(ss[j >> 2], head_lane(j)) * (double)nw);
        t[j] = q[j] * q[j];
        if (j < H_idx) c = fma(0.5 * (double)readlane_f(al_l, j), (double)q[j], c);
      }
      wave_sums_butterfly_f<HM>(t, n2);
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        n2[i] = sqrtf(n2[i]) * 1.0001f;
        sc[i] = score_scale(n2[i]);
      }
#pragma unroll
      for (int j = 0; j < HM; ++j) {
        const float f = readlane_f(sc[j >> 2], head_lane(j));
        const _Float16 hv = score_half(q[j] * f);
        const float r = q[j] * f - (float)hv;
        t[j] = r * r;
        if (j < H_idx) *(_Float16*)(sb + j * SB::HEAD + place) = hv;
      }
      wave_sums_butterfly_f<HM>(t, r2);
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int j = 4 * i + 2 * (rho & 1) + (rho >> 1);
        const float al = __shfl(al_l, j);
        if (holds && j < H_idx) {
          const float a = 0.5f * al / sc[i];
          sane = sane && score_sane(al) && score_sane(n2[i]);
          err += fabsf(a) * (1.001f * sqrtf(r2[i]) + 0x1p-16f * n2[i] * sc[i]);
          rows[j * 16 + m] = a;
        }
      }
      err = wave_sum_f(err);
    } else {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int j = i * HP + hl;
        const bool on = j < H_idx;
        const float al = on ? __shfl(al_l, j) : 0.f;
        const double rr = sqrt(row16_sum_d(v[i] * v[i]) / (double)DI + (double)rms_eps);
        q[i] = (float)(v[i] / rr * (double)nw);
        const float norm = sqrtf(row16_sum_f(q[i] * q[i])) * 1.0001f, f = score_scale(norm);
        const _Float16 hv = score_half(q[i] * f);
        const float r = q[i] * f - (float)hv;
        const float a = 0.5f * al / f, r2 = row16_sum_f(r * r);
        if (on) {
          sane = sane && score_sane(al) && score_sane(norm);
          err += fabsf(a) * (1.001f * sqrtf(r2) + 0x1p-16f * norm * f);
          c = fma(0.5 * (double)al, (double)q[i], c);
          *(_Float16*)(sb + j * SB::HEAD + place) = hv;
          if (d == 0) rows[j * 16 + m] = a;
        }
      }
      c = rows_sum_d(c);
      err = rows_sum_f(err);
    }
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (i * HP + hl < H_idx) qf[(row * H_idx + i * HP + hl) * DI + d] = q[i];
    const float cf = (float)c;
    float c2 = cf * cf;
    if constexpr (DI == 64) c2 = wave_sum_f(c2); else c2 = row16_sum_f(c2);
    const float cn = sqrtf(c2) * 1.0001f, f = score_scale(cn);
    const _Float16 hv = score_half(cf * f);
    const float r = (float)(c * (double)f - (double)(float)hv);
    float r2 = r * r;
    if constexpr (DI == 64) r2 = wave_sum_f(r2); else r2 = row16_sum_f(r2);
    sane = sane && score_sane(cn);
    err += (1.001f * sqrtf(r2) + 0x1p-16f * cn * f) / f;
    // (err is at least 2^-16 of what the sum of the heads' terms can reach: below 2^80 no part of that sum is infinite, and an
    // infinity of either sign cannot meet one of the other)
    sane = __all(sane && err < 0x1p80f);
    if (lane < DI) *(_Float16*)(sb + HM * SB::HEAD + place) = sane ? hv : (_Float16)0.f;
    if (!sane) {   // (operands of zero: infinities and NaN stay out of the sum, whose bound is then infinite)
      for (int j = hl; j < H_idx; j += HP) {
        *(_Float16*)(sb + j * SB::HEAD + place) = (_Float16)0.f;
        if (d == 0) rows[j * 16 + m] = 0.f;
      }
    }
    if (lane == 0) {
      rows[SB::T * 16 + m] = sane ? 1.f / f : 0.f;
      rows[SB::ERR * 16 + m] = sane ? 1.01f * 4096.f * err : INFINITY;   // out of range: always a candidate
      ((int*)rows)[SB::POS * 16 + m] = my_pos;
    }
  }
  __syncthreads();
  uint4* dst = (uint4*)(blocks + ((size_t)b * gridDim.x + blockIdx.x) * SB::BYTES);
  for (int i = tid; i < SB::BYTES / 16; i += 1024) dst[i] = ((const uint4*)sb)[i];
}

// a key's fp16 operand for one lane (dims DPL kq .. of the key), scaled so that the key's norm is in [2^11, 2^12).
// A key with infinities, NaN or a norm of 2^100 has no bounds: its scale and its products are NaN, and every query is a
// candidate.
template <int DI>
struct ScoreKey {
  im_h8 h[DI == 64 ? 2 : 1];   // (DI = 16: 4 values, in the lower half)
  float scale;
};
template <int DI>
__device__ __forceinline__ ScoreKey<DI> score_key_operand(const bf16_t* __restrict__ krow, int kq) {
  ScoreKey<DI> o;
  float f[DI / 4];
  if constexpr (DI == 64) {
    const uint4 u0 = *(const uint4*)(krow + 16 * kq), u1 = *(const uint4*)(krow + 16 * kq + 8);
    const uint32_t u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) { f[2 * i] = bf_lo(u[i]); f[2 * i + 1] = bf_hi(u[i]); }
  } else {
    const uint2 u = *(const uint2*)(krow + 4 * kq);
    f[0] = bf_lo(u.x); f[1] = bf_hi(u.x); f[2] = bf_lo(u.y); f[3] = bf_hi(u.y);
  }
  float n2 = 0.f;
#pragma unroll
  for (int i = 0; i < DI / 4; ++i) n2 = fmaf(f[i], f[i], n2);
  const float norm = sqrtf(rows_sum_f(n2)) * 1.0001f;
  o.scale = norm < 0x1p100f ? score_scale(norm) : NAN;
  if constexpr (DI == 16) {
#pragma unroll
    for (int i = 4; i < 8; ++i) o.h[0][i] = (_Float16)0.f;
  }
#pragma unroll
  for (int i = 0; i < DI / 4; ++i) o.h[i / 8][i % 8] = score_half(f[i] * o.scale);   // (NaN stays NaN)
  return o;
}

// z[query 4 kq + r][key l16] of one head: DI contracted dims
template <int DI>
__device__ __forceinline__ im_f4 score_product(const char* head, int lane, const ScoreKey<DI>& k) {
  const im_f4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (DI == 64) {
    const im_h8 a0 = *(const im_h8*)(head + lane * 16), a1 = *(const im_h8*)(head + 1024 + lane * 16);
    const im_f4 z = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, k.h[0], zero, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, k.h[1], z, 0, 0, 0);
  } else {
    const im_h4 a0 = *(const im_h4*)(head + lane * 8);
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a0, __builtin_shufflevector(k.h[0], k.h[0], 0, 1, 2, 3), zero, 0, 0, 0);
  }
}

// grid (ceil(max_live / (64 TPW)) * units, groups), 4 waves; a wave owns TPW tiles of 16 keys, their fp16 operands in
// registers, and the workgroup walks over the query blocks (two LDS buffers, the next block on its way while one is
// in use), from the last one down to the first that sees the tile: every resident workgroup then reads the
// same blocks at about the same time, so they come from the XCD's L2.  Tiles of low slots see the most queries: they
// are dispatched first.  grid y: groups of blocks_per_group query blocks (short caches), each with records of its own.
// Bound by the matrix cores at the clock that the power leaves them: 1.62 GHz, and 70 % of the cycles have a product
// (counters; 4 x 16384 tokens, 8 heads: 4.2 ms, fp64 products of all pairs 76.8).  8 tiles per wave, with half the LDS reads
// per product, took the same time (4.35 ms).
// Record [group][unit][key][kq]: over the queries 4 kq .. 4 kq + 3 of every block, (u1, u2) = largest and second
// largest of the blocks' maxima of the upper bound, i1 = block of u1.
template <int DI, int HM, int TPW>
__global__ __launch_bounds__(256, HM == 8 ? 4 : 2) void k_score_scan(const bf16_t* __restrict__ Kidx, const int32_t* __restrict__ pos,
                                                       const int32_t* __restrict__ len,
                                                       int32_t* __restrict__ n_projected,
                                                       const char* __restrict__ blocks,
                                                       const int32_t* __restrict__ q_pos, int n_q, int sets_per_b, int C,
                                                       int H_idx, int max_live, int units, int blocks_per_group,
                                                       int rec_live, float2* __restrict__ rec_u,
                                                       int32_t* __restrict__ rec_i) {
  using SB = ScoreBlock<DI, HM>;
  __shared__ __attribute__((aligned(16))) char sq[2][SB::BYTES];
  __shared__ int s_min[4], s_first[4];
  const int unit = blockIdx.x % units, tile = blockIdx.x / units;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = unit / sets_per_b;
  const int n = min(len[unit], max_live);
  if (tile == 0 && blockIdx.y == 0 && tid == 0) n_projected[unit] = n;  // the projection kernel ran before
  const int t0 = tile * (64 * TPW);
  if (t0 >= n) return;
  const int kbase = t0 + 16 * TPW * w;
  ScoreKey<DI> key[TPW];
  int posk[TPW];
  int mn = INT_MAX, mx = INT_MIN, wild = 0;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {   // (keys past the end repeat the last live one; their records are not written)
    const int k = min(kbase + 16 * t + l16, n - 1);
    key[t] = score_key_operand<DI>(Kidx + ((size_t)unit * C + k) * DI, kq);
    posk[t] = pos[(size_t)unit * C + k];
    wild |= (key[t].scale != key[t].scale) ? 1 << t : 0;
    mn = min(mn, posk[t]);
    mx = max(mx, posk[t]);
  }
  mn = (int)(wave_min_u((uint32_t)mn ^ 0x80000000u) ^ 0x80000000u);
  mx = (int)(wave_max_u((uint32_t)mx ^ 0x80000000u) ^ 0x80000000u);
  // the first query that sees any key of the tile: no query before it does
  if (lane == 0) s_min[w] = mn;
  __syncthreads();
  const int tile_min = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
  const int32_t* qp_b = q_pos + (size_t)b * n_q;
  int first = n_q;
  for (int i = tid; i < n_q; i += 256)
    if (qp_b[i] >= tile_min) { first = i; break; }
  first = (int)wave_min_u((uint32_t)first);
  if (lane == 0) s_first[w] = first;
  __syncthreads();
  first = min(min(s_first[0], s_first[1]), min(s_first[2], s_first[3]));
  const int nblk = (n_q + 15) / 16;
  const int b_lo = max((int)blockIdx.y * blocks_per_group, first / 16);
  const int b_hi = min(nblk, ((int)blockIdx.y + 1) * blocks_per_group);
  const char* src = blocks + (size_t)b * nblk * SB::BYTES;

  float u1[TPW], u2[TPW];
  int i1[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) { u1[t] = u2[t] = -INFINITY; i1[t] = 0; }
  auto fetch = [&](int blk, int buf) {
    for (int c = w; c < SB::BYTES / 1024; c += 4)
      copy_to_lds_1k(src + (size_t)blk * SB::BYTES + c * 1024 + lane * 16, &sq[buf][c * 1024]);
  };
  if (b_hi > b_lo) fetch(b_hi - 1, 0);
  int buf = 0;
#pragma unroll 1
  for (int blk = b_hi - 1; blk >= b_lo; --blk, buf ^= 1) {
    copy_wait<0>();                                     // this wave's part of the block has arrived
    __syncthreads();                                    // ... and everyone's; the other buffer is free again
    if (blk > b_lo) fetch(blk - 1, buf ^ 1);
    const char* q = sq[buf];
    const float* rows = (const float*)(q + SB::OFF);
    const im_f4 t4 = *(const im_f4*)(rows + SB::T * 16 + 4 * kq), e4 = *(const im_f4*)(rows + SB::ERR * 16 + 4 * kq);
    const int4 qp = *(const int4*)(rows + SB::POS * 16 + 4 * kq);
    im_f4 acc[TPW];
    {
      im_f4 z[TPW];
#pragma unroll
      for (int t = 0; t < TPW; ++t) z[t] = score_product<DI>(q + HM * SB::HEAD, lane, key[t]);
#pragma unroll
      for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t][r] = fmaf(t4[r], z[t][r], e4[r]);
    }
#pragma unroll 1
    for (int j0 = 0; j0 < H_idx; j0 += 2) {   // (an absent head's operands and a_j are zero)
#pragma unroll
      for (int j = j0; j < j0 + 2; ++j) {
        const im_f4 a4 = *(const im_f4*)(rows + j * 16 + 4 * kq);
        im_f4 z[TPW];
#pragma unroll
        for (int t = 0; t < TPW; ++t) z[t] = score_product<DI>(q + j * SB::HEAD, lane, key[t]);
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[t][r] = fmaf(a4[r], fabsf(z[t][r]), acc[t][r]);
      }
    }
    if (!__all(min(min(qp.x, qp.y), min(qp.z, qp.w)) >= mx)) {   // some query does not see some key of the wave
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        acc[t][0] = (qp.x >= posk[t]) ? acc[t][0] : -INFINITY;
        acc[t][1] = (qp.y >= posk[t]) ? acc[t][1] : -INFINITY;
        acc[t][2] = (qp.z >= posk[t]) ? acc[t][2] : -INFINITY;
        acc[t][3] = (qp.w >= posk[t]) ? acc[t][3] : -INFINITY;
      }
    }
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const float m = fmaxf(fmaxf(acc[t][0], acc[t][1]), fmaxf(acc[t][2], acc[t][3]));
      i1[t] = (m > u1[t]) ? blk : i1[t];
      u2[t] = __builtin_amdgcn_fmed3f(m, u1[t], u2[t]);
      u1[t] = fmaxf(u1[t], m);
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int k = kbase + 16 * t + l16;
    if (k < n) {
      const size_t at = (((size_t)blockIdx.y * units + unit) * rec_live + k) * 4 + kq;
      if ((wild >> t & 1) && b_hi > b_lo) { u1[t] = u2[t] = INFINITY; i1[t] = b_lo; }   // (its maxima were of NaN)
      rec_u[at] = make_float2(u1[t], u2[t]);
      rec_i[at] = i1[t];
    }
  }
}

// grid (ceil(max_live / (4 KPW)), units), 4 waves of KPW keys each (16, or 4).  A candidate is a record's block: its 4 queries are
// evaluated in fp64 by the whole wave (lane (query r = lane / 16, p): dims 4 p .. of every head).  Bound by the vector
// ALU: half of it conversions and products, half the sums over 16 lanes, which is why the heads' sums are taken together.  A
// second candidate block inside one record is not known by name: the key goes to the list.  So do all keys of a wave whose
// candidates number more than IM_EXACT_NAMED per key (queries that are equal, or gates of zero): the list takes whole blocks
// through the fp64 matrix cores, from the best of what was evaluated.  64 equal queries x 65536 keys x 8 heads, the call: 449 us
// without this, with 2, 3 and 4 candidates 253, 261 and 281; with gates of zero 429, 180, 164 and 182.
#define IM_EXACT_NAMED 4
template <int DI, int HM>
__device__ __forceinline__ float score_exact4(const float* __restrict__ qrow, const float* __restrict__ al, int H_idx,
                                              const float* kd, int p) {
  constexpr int PD = DI / 16;
  const bool b3 = p & 8, b2 = p & 4, b1 = p & 2;
  const int head = p >> 1;   // of 8, whose sum ends in this lane
  auto pick = [](bool b, double lo, double hi) { return b ? hi : lo; };   // (of values: of array elements it is an indexed load)
  double acc = 0.0;
#pragma unroll
  for (int j0 = 0; j0 < HM; j0 += 8) {
    if (j0 >= H_idx) break;
    float qv[8][PD];   // (heads past the last repeat it, unused)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = min(j0 + i, H_idx - 1);
      if constexpr (PD == 4) {
        const float4 t = *(const float4*)(qrow + j * DI + 4 * p);
        qv[i][0] = t.x; qv[i][1] = t.y; qv[i][2] = t.z; qv[i][3] = t.w;
      } else {
        qv[i][0] = qrow[j * DI + p];
      }
    }
    const float av = al[j0 + head];
    double z[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      z[i] = 0.0;
#pragma unroll
      for (int m = 0; m < PD; ++m) z[i] = fma((double)qv[i][m], (double)kd[m], z[i]);
    }
    // the 8 heads' sums over the 16 lanes: after each step a lane goes on with half of the heads
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] += dpp_zero_d<0x128, 0xF>(z[i]);                                    // lane ^ 8
#pragma unroll
    for (int i = 0; i < 4; ++i) { z[i] = pick(b3, z[i], z[i + 4]); z[i] += dpp_zero_d<0x141, 0xF>(z[i]); }   // lane ^ 7
#pragma unroll
    for (int i = 0; i < 2; ++i) { z[i] = pick(b2, z[i], z[i + 2]); z[i] += dpp_zero_d<0x4E, 0xF>(z[i]); }    // lane ^ 2
    z[0] = pick(b1, z[0], z[1]);
    z[0] += dpp_zero_d<0xB1, 0xF>(z[0]);                                                                 // lane ^ 1
    if (j0 + head < H_idx) acc = fma((double)av, fmax(z[0], 0.0), acc);
  }
  acc += dpp_zero_d<0x4E, 0xF>(acc);     // over the heads
  acc += dpp_zero_d<0x141, 0xF>(acc);
  acc += dpp_zero_d<0x128, 0xF>(acc);
  return (float)acc;
}
// this lane's share (dims PD p ..) of a key
template <int DI>
__device__ __forceinline__ void score_exact_key(const bf16_t* __restrict__ krow, float* kd, int p) {
  if constexpr (DI == 64) {
    const uint2 u = *(const uint2*)(krow + 4 * p);
    kd[0] = bf_lo(u.x); kd[1] = bf_hi(u.x); kd[2] = bf_lo(u.y); kd[3] = bf_hi(u.y);
  } else {
    kd[0] = bf2f(krow[p]);
  }
}

template <int DI, int HM, int KPW>
__global__ __launch_bounds__(256) void k_score_exact(const bf16_t* __restrict__ Kidx, const int32_t* __restrict__ pos,
                                                     const int32_t* __restrict__ len, const char* __restrict__ blocks,
                                                     const float* __restrict__ qf, const float* __restrict__ al16,
                                                     const int32_t* __restrict__ q_pos, int n_q, int sets_per_b, int C,
                                                     int H_idx, int max_live, int groups, int rec_live,
                                                     const float2* __restrict__ rec_u, const int32_t* __restrict__ rec_i,
                                                     float* __restrict__ scores, int32_t* __restrict__ n_listed,
                                                     int2* __restrict__ listed) {
  using SB = ScoreBlock<DI, HM>;
  constexpr int PD = DI / 16;
  const int unit = blockIdx.y, units = gridDim.y, b = unit / sets_per_b;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int n = min(len[unit], max_live);
  const int kbase = (blockIdx.x * 4 + w) * KPW;
  if (kbase >= n) return;
  const bool mine = l16 < KPW && kbase + l16 < n;
  const int key = mine ? kbase + l16 : kbase, nblk = (n_q + 15) / 16;
  const int pk = pos[(size_t)unit * C + key];
  float u1[IM_SCORE_GROUPS], u2[IM_SCORE_GROUPS], lmax = -INFINITY;
  int i1[IM_SCORE_GROUPS], ib = 0;
#pragma unroll
  for (int g = 0; g < IM_SCORE_GROUPS; ++g) {
    u1[g] = u2[g] = -INFINITY;
    i1[g] = 0;
    if (g < groups) {
      const size_t at = (((size_t)g * units + unit) * rec_live + key) * 4 + kq;
      const float2 u = rec_u[at];
      u1[g] = u.x; u2[g] = u.y;
      i1[g] = rec_i[at];
      if (u1[g] > lmax) { lmax = u1[g]; ib = i1[g]; }
    }
  }
  const float top = rows_max_f(lmax);   // the key's largest upper bound
  float err = -INFINITY;
  if (lmax == top && top > -INFINITY) {
    const float4 e4 = *(const float4*)(blocks + ((size_t)b * nblk + ib) * SB::BYTES + SB::OFF + (SB::ERR * 16 + 4 * kq) * 4);
    err = fmaxf(fmaxf(e4.x, e4.y), fmaxf(e4.z, e4.w));
  }
  err = rows_max_f(err);
  // the maximal score (in the bounds' scale) is at least this
  const float low = (top == INFINITY) ? -INFINITY : top - 2.001f * err - 0x1p-18f * fabsf(top);
  float best = -INFINITY;
  bool more = false;
  int room = IM_EXACT_NAMED * KPW;   // (uniform)
#pragma unroll
  for (int g = 0; g < IM_SCORE_GROUPS; ++g) {
    if (g >= groups) break;
    more = more || (u2[g] >= low && u2[g] > -INFINITY);
    unsigned long long cand = __ballot(mine && u1[g] >= low && u1[g] > -INFINITY);
    while (cand) {
      if (--room < 0) break;
      const int ln = __builtin_ctzll(cand);
      cand &= cand - 1;
      const int blk = __builtin_amdgcn_readlane(i1[g], ln), kk = ln & 15;
      const int pkk = __builtin_amdgcn_readlane(pk, ln);
      const int s = 16 * blk + 4 * (ln >> 4) + kq, sc = min(s, n_q - 1);
      const size_t row = (size_t)b * n_q + sc;
      float kd[PD];
      score_exact_key<DI>(Kidx + ((size_t)unit * C + kbase + kk) * DI, kd, l16);
      const int qp = q_pos[row];
      const float v = score_exact4<DI, HM>(qf + row * H_idx * DI, al16 + row * 16, H_idx, kd, l16);
      const float m = rows_max_f((s < n_q && qp >= pkk) ? v : -INFINITY);
      if (l16 == kk) best = fmaxf(best, m);
    }
  }
  more = rows_max_f(more || (room < 0 && lmax > -INFINITY) ? 1.f : 0.f) > 0.f && mine;
  if (kq == 0 && mine) scores[(size_t)unit * C + key] = best;
  const unsigned long long lst = __ballot(more && kq == 0);
  if (lst) {
    int base = 0;
    if (lane == 0) base = atomicAdd(n_listed + b, __popcll(lst));
    base = __builtin_amdgcn_readfirstlane(base);
    if (more && kq == 0)
      listed[(size_t)b * sets_per_b * C + base + __popcll(lst & ((1ull << lane) - 1ull))] = make_int2(unit, key);
  }
}

// A fixed number of workgroups over the listed keys.  An item is 64 keys of one sequence (16 per wave) against a
// segment of its query blocks; the segments are as short as fills the grid, and not below IM_LIST_BLOCKS.
// scores[key] rises by atomic maxima; reading an older value only costs work.  (Segments of 8 blocks at least: 562
// queries 20 us, of 2: 14.)
#define IM_LIST_WGS 1024
#define IM_LIST_BLOCKS 2
template <int DI, int HM>
__global__ __launch_bounds__(256, HM == 8 ? 4 : 2) void k_score_listed(const bf16_t* __restrict__ Kidx,
                                                                       const int32_t* __restrict__ pos,
                                                                       const char* __restrict__ blocks,
                                                                       const float* __restrict__ qf,
                                                                       const float* __restrict__ al16, int B, int n_q,
                                                                       int sets_per_b, int C, int H_idx,
                                                                       float* __restrict__ scores,
                                                                       const int32_t* __restrict__ n_listed,
                                                                       const int2* __restrict__ listed) {
  using SB = ScoreBlock<DI, HM>;
  constexpr int DPL = DI / 4;
  __shared__ __attribute__((aligned(16))) char sq[2][SB::BYTES];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nblk = (n_q + 15) / 16;
  long long chunks = 0;
  for (int b = 0; b < B; ++b) chunks += (n_listed[b] + 63) / 64;
  if (chunks == 0) return;
  int segs = (int)min((2 * IM_LIST_WGS + chunks - 1) / chunks, (long long)((nblk + IM_LIST_BLOCKS - 1) / IM_LIST_BLOCKS));
  const int per_seg = (nblk + segs - 1) / segs;
  segs = (nblk + per_seg - 1) / per_seg;
  int b = 0;
  long long before = 0;                                    // items of the sequences before b
  for (long long item = blockIdx.x; item < chunks * segs; item += gridDim.x) {   // (ascending, so b ascends)
    int cnt = n_listed[b];
    while (item >= before + (long long)((cnt + 63) / 64) * segs) {
      before += (long long)((cnt + 63) / 64) * segs;
      cnt = n_listed[++b];
    }
    const int k0 = (int)((item - before) / segs) * 64 + 16 * w, seg = (int)((item - before) % segs);
    const int2 uk = listed[(size_t)b * sets_per_b * C + min(k0 + l16, cnt - 1)];   // (past the end: the last one again)
    const size_t at = (size_t)uk.x * C + uk.y;
    const ScoreKey<DI> key = score_key_operand<DI>(Kidx + at * DI, kq);
    const int pk = pos[at];
    const float start = scores[at];
    float best = start;
    const int b_lo = seg * per_seg, b_hi = min(nblk, b_lo + per_seg);
    const char* src = blocks + (size_t)b * nblk * SB::BYTES;
    auto fetch = [&](int blk, int buf) {
      for (int c = w; c < SB::BYTES / 1024; c += 4)
        copy_to_lds_1k(src + (size_t)blk * SB::BYTES + c * 1024 + lane * 16, &sq[buf][c * 1024]);
    };
    __syncthreads();                                       // (the item before is done with the buffers)
    fetch(b_lo, 0);
    int buf = 0;
#pragma unroll 1
    for (int blk = b_lo; blk < b_hi; ++blk, buf ^= 1) {
      copy_wait<0>();
      __syncthreads();
      if (blk + 1 < b_hi) fetch(blk + 1, buf ^ 1);
      const char* q = sq[buf];
      const float* rows = (const float*)(q + SB::OFF);
      const im_f4 t4 = *(const im_f4*)(rows + SB::T * 16 + 4 * kq), e4 = *(const im_f4*)(rows + SB::ERR * 16 + 4 * kq);
      const int4 qp = *(const int4*)(rows + SB::POS * 16 + 4 * kq);
      im_f4 z = score_product<DI>(q + HM * SB::HEAD, lane, key), acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = fmaf(t4[r], z[r], e4[r]);
#pragma unroll 1
      for (int j0 = 0; j0 < H_idx; j0 += 4) {   // (absent heads' operands and a_j are zero)
        im_f4 a4[4], zz[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a4[i] = *(const im_f4*)(rows + (j0 + i) * 16 + 4 * kq);
          zz[i] = score_product<DI>(q + (j0 + i) * SB::HEAD, lane, key);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r] = fmaf(a4[i][r], fabsf(zz[i][r]), acc[r]);
      }
      // (a finite score may be infinite in the bounds' units: an infinite bound stays above it)
      const float bar = (best == INFINITY) ? INFINITY : fminf(best * key.scale, 3.402823466e38f);
      // (negated: a key without bounds is a hit)
      const bool hit = (qp.x >= pk && !(acc[0] <= bar)) || (qp.y >= pk && !(acc[1] <= bar)) ||
                       (qp.z >= pk && !(acc[2] <= bar)) || (qp.w >= pk && !(acc[3] <= bar));
      unsigned long long hits = __ballot(hit);
      if (!hits) continue;
      if (__popcll(hits) <= 4) {   // (usual) lane by lane: its 4 queries against its key, as k_score_exact does it
        while (hits) {
          const int ln = __builtin_ctzll(hits);
          hits &= hits - 1;
          const int unit = __builtin_amdgcn_readlane(uk.x, ln), slot = __builtin_amdgcn_readlane(uk.y, ln);
          const int pkk = __builtin_amdgcn_readlane(pk, ln);
          const int s = 16 * blk + 4 * (ln >> 4) + kq;
          const size_t row = (size_t)b * n_q + min(s, n_q - 1);
          float kd[DI / 16];
          score_exact_key<DI>(Kidx + ((size_t)unit * C + slot) * DI, kd, l16);
          const float v = score_exact4<DI, HM>(qf + row * H_idx * DI, al16 + row * 16, H_idx, kd, l16);
          const int qps = ((const int*)rows)[SB::POS * 16 + 4 * (ln >> 4) + kq];
          const float m = rows_max_f((s < n_q && qps >= pkk) ? v : -INFINITY);
          if (l16 == (ln & 15)) best = fmaxf(best, m);
        }
        continue;
      }
      // fp64 for the whole 16 x 16 block: rows = queries (lane (l16, kq) supplies dims DPL kq .. of query l16), columns
      // = keys; result register r is query 4 r + kq, key l16
      double kd[DPL];
      if constexpr (DI == 64) {
        const uint4 u0 = *(const uint4*)(Kidx + at * DI + 16 * kq), u1 = *(const uint4*)(Kidx + at * DI + 16 * kq + 8);
        const uint32_t u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) { kd[2 * i] = (double)bf_lo(u[i]); kd[2 * i + 1] = (double)bf_hi(u[i]); }
      } else {
        const uint2 u = *(const uint2*)(Kidx + at * DI + 4 * kq);
        kd[0] = (double)bf_lo(u.x); kd[1] = (double)bf_hi(u.x); kd[2] = (double)bf_lo(u.y); kd[3] = (double)bf_hi(u.y);
      }
      const size_t row0 = (size_t)b * n_q + 16 * blk;
      const float* qr = qf + (row0 + min(l16, n_q - 1 - 16 * blk)) * H_idx * DI + DPL * kq;
      double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int j = 0; j < H_idx; ++j) {
        im_v4d zd = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int m = 0; m < DPL; m += 4) {
          const float4 t = *(const float4*)(qr + j * DI + m);
          zd = __builtin_amdgcn_mfma_f64_16x16x4f64((double)t.x, kd[m], zd, 0, 0, 0);
          zd = __builtin_amdgcn_mfma_f64_16x16x4f64((double)t.y, kd[m + 1], zd, 0, 0, 0);
          zd = __builtin_amdgcn_mfma_f64_16x16x4f64((double)t.z, kd[m + 2], zd, 0, 0, 0);
          zd = __builtin_amdgcn_mfma_f64_16x16x4f64((double)t.w, kd[m + 3], zd, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int s = min(4 * r + kq, n_q - 1 - 16 * blk);
          s4[r] = fma((double)al16[(row0 + s) * 16 + j], fmax(zd[r], 0.0), s4[r]);
        }
      }
      float m = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int qpr = ((const int*)rows)[SB::POS * 16 + 4 * r + kq];
        if (16 * blk + 4 * r + kq < n_q && qpr >= pk) m = fmaxf(m, (float)s4[r]);
      }
      best = fmaxf(best, rows_max_f(m));
    }
    if (kq == 0 && k0 + l16 < cnt && best > start) {
      // fp32 maximum by integer atomics: the bit patterns of positive numbers ascend, of negative ones descend (-0.0 is one
      // of these, the least: a score of -1e-50 rounds to it)
      if (__float_as_int(best) >= 0) atomicMax((int*)(scores + at), __float_as_int(best));
      else atomicMin((unsigned*)(scores + at), __float_as_uint(best));
    }
  }
}
