// Fused decode step: the whole path for one new token per sequence in three launches.
//   k_dec_prep   : the roles that do not need each other's results: append of the new (k, v), its indexer key, the
//                  query-side indexer projections (U_q, G; head-shared layout: U_k, too), the terms of the memory
//                  readout that do not depend on this step's eviction (phi_q, phi_q^T M, phi_q^2 . b, gate).
//   k_dec_score  : workgroups that score keys in fp64 (every wave leaves the last-ranked entry of its own), and split workgroups,
//                  which stream K and V of 128 keys each and leave softmax-attention partials.
//   k_dec_finish : the last-ranked entry of all, merge of the partials without it, gated readout; a unit's workgroups
//                  share the memory update, and the last of them to have read the cache fills the hole.
// Steps that score nothing (attention only, or the slot to evict is named by the caller) take two: the split workgroups run beside
// the roles of the first (k_dec_attend).
// Head-shared layout: one indexer key per token, one decision and one memory per sequence; the same kernels.
//
// A launch boundary is the cheapest dependency between workgroups here (a device-scope release, an L2 write-back,
// per workgroup or an in-kernel wait costs several microseconds more than a launch).  Two are needed: scores need the projections of all
// workgroups, the output needs the decision over all keys.  The stream of K and V needs neither; it runs beside the scores, whose
// chain (7 us as a launch of its own) it hides.  A part of it in the first launch does not pay: 4 tokens x 8 layers of 4 x 2048 entries
// with none, a quarter, half, all of the splits there 746, 780, 795, 810 us, of 1 x 4096 619, 662, 656, 638.
// Split and scoring workgroups are different ones, so the decision is not known to a partial: it holds all of its keys, and
// k_dec_finish takes the evicted one out again.  With the roles as waves of one workgroup that met at a barrier, every split left its
// last-ranked entry out and wrote it to a record, and the last launch staged all records: 23.9 us a layer-step of 4 x 2048 entries x
// 8 heads, 22.8 now (1 x 4096: 21.4, 18.2; 8 x 1024 with index reuse over four layers: 20.7, 18.0; head-shared 4 x 2048, with a
// launch of its own for the scores: 26.8, 20.2).
// Same results as append -> index_score (n_q = 1) -> topb_select -> memory_update -> compact_kv
// -> decode_attn_with_readout whenever every unit enters with len <= budget.
#pragma once
#include <type_traits>

#include "im_device.h"

#define DEC_KEYS 128                 // keys per split workgroup (4 waves of 32)
#define DEC_GMAX 8                   // query heads per KV head supported
// The counters of k_dec_finish lie on cache lines of their own (in 32-bit words): arrivals at one line are taken one after another, also
// at different counters.  256 workgroups, all counters on one or two lines / one a line, us per layer-step (an index-reuse
// follower): head-shared 4 x 2048, 8 x 8 heads 18.6 / 17.3, 8 x 1024, 4 x 8 heads 17.7 / 16.6; per-unit 4 x 2048, 8 x 8 heads 17.1 / 16.5
#define DEC_LINE 32

typedef double v4d __attribute__((ext_vector_type(4)));

struct DecArgs {
  // state
  bf16_t *K, *V, *Kidx;
  int32_t *pos, *len, *nproj;
  float *M, *bvec;
  // slow weights
  const bf16_t *Uq, *Gw, *Uk, *nqw, *nkw, *Wt, *wg;
  float cg;
  // inputs
  const bf16_t *q, *xg, *k_new, *v_new;
  const int32_t *pos_new, *q_pos;
  const int32_t* named;   // optional [sets]: the slot to evict is given by the caller (-1 or >= len: none)
  // outputs
  bf16_t* out;
  float* readout;
  float* scores;      // optional
  int32_t* evicted;   // optional
  // workspace
  double *qy, *alpha;   // U_q q, G x
  double* xk;           // head-shared layout: U_k x of the new token, [B][16]
  int32_t *status, *maxpos;
  int32_t* arrived;     // [sets * DEC_LINE] workgroups of k_dec_finish that are done with the cache
  float* part;          // [units][S][G][128] numerators
  float2* part_ml;      // [units][S][G] maximum, denominator
  float* qm;            // per unit: the eviction-independent terms of the memory readout (DEC_QM floats per head)
  uint4* pick;          // [sets][n_pick] last-ranked entry of each wave of k_dec_score (rank key hi, lo, slot or -1)
  // scalars
  int B, H, H_kv, G, C, H_idx, gate_in, n_sink, n_recent, budget, S, max_live;
  uint32_t kv_magic;    // floor(2^32 / H_kv) + 1: the high word of u * kv_magic is u / H_kv (u < 2^16, H_kv > 1)
  int score;            // the step scores its keys (else: attention only, or the slot is named)
  int n_pick;           // waves of k_dec_score per set (0: nothing is scored)
  int n_proj;           // projection blocks
  // head-shared layout (hs = 1): the H_set = H_kv units of a sequence form one set; len, pos, Kidx
  // (di = 16 values per row), nproj, M, bvec are indexed by the set u / H_set.  Else H_set = 1, di = 64.
  int hs, H_set, di;
  float rms_eps, mem_eps, scale, lambda, eta;
  double alpha_denom;   // sqrt(H_idx di)
};

// wait until at most 4 of this wave's vector memory loads are outstanding (loads return in order)
__device__ __forceinline__ void dec_pace4() { asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); }

__device__ __forceinline__ void unpack8(const uint4& u, float* f) {
  f[0] = bf_lo(u.x); f[1] = bf_hi(u.x); f[2] = bf_lo(u.y); f[3] = bf_hi(u.y);
  f[4] = bf_lo(u.z); f[5] = bf_hi(u.z); f[6] = bf_lo(u.w); f[7] = bf_hi(u.w);
}

// --------------------------------------------------------------------------------------------
// Roles of the first launch
// --------------------------------------------------------------------------------------------
// out_rows[m][r] = sum_k A[m][k] Bm[n0 + r][k] for r = 0, 1 and every batch row m (bf16 inputs, fp64
// accumulation).  Each round issues the loads of two 2048-wide slabs before any arithmetic.
template <int MB>
__device__ __forceinline__ void dec_gemv2(const bf16_t* __restrict__ A, const bf16_t* __restrict__ Bm, int n0,
                                          int N, int M, int Kd, double (*part)[16], double* out_rows,
                                          int m_first = 0, int m_end = 1 << 30) {
  const int tid = threadIdx.x;
  const int r1 = (n0 + 1 < N) ? n0 + 1 : n0;   // an absent second row repeats the first (result unused)
  m_end = min(m_end, M);                       // batch rows [m_first, m_end) only
  for (int mb = m_first; mb < m_end; mb += MB) {
    double acc[MB][2];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i][0] = acc[i][1] = 0.0;
    for (int k0 = tid * 8; k0 < Kd; k0 += 2 * 2048) {
      uint4 bu[2][2], au[2][MB];
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int k = (k0 + it * 2048 < Kd) ? k0 + it * 2048 : k0;
        bu[it][0] = *(const uint4*)(Bm + (size_t)n0 * Kd + k);
        bu[it][1] = *(const uint4*)(Bm + (size_t)r1 * Kd + k);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const int m = (mb + i < M) ? mb + i : M - 1;
          au[it][i] = *(const uint4*)(A + (size_t)m * Kd + k);
        }
      }
      // MB = 4: every load above is issued before the arithmetic starts.  The empty statement needs a word of
      // each, and nothing is scheduled across the barrier; else the second slab's loads sink into its branch
      // below and their latency is paid a second time.  (With 8 batch rows the registers this takes would
      // halve the number of resident workgroups.)
      if constexpr (MB == 4) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(bu[0][0].x), "+v"(bu[0][1].x), "+v"(bu[1][0].x), "+v"(bu[1][1].x),
                          "+v"(au[0][0].x), "+v"(au[0][1].x), "+v"(au[0][2].x), "+v"(au[0][3].x),
                          "+v"(au[1][0].x), "+v"(au[1][1].x), "+v"(au[1][2].x), "+v"(au[1][3].x));
      }
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        if (k0 + it * 2048 < Kd) {
          float b0[8], b1[8];
          unpack8(bu[it][0], b0);
          unpack8(bu[it][1], b1);
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            float av[8];
            unpack8(au[it][i], av);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              acc[i][0] = fma((double)av[e], (double)b0[e], acc[i][0]);
              acc[i][1] = fma((double)av[e], (double)b1[e], acc[i][1]);
            }
          }
        }
      }
    }
    // the 2 MB wave sums as one butterfly (value 2 i + r = batch row i, weight row r), then the 4 waves
    // meet in LDS: lane 15 of row rho of register i holds value 4 i + 2 (rho & 1) + (rho >> 1)
    double ws[MB / 2];
    wave_sums_butterfly_d<2 * MB>(&acc[0][0], ws);
    __syncthreads();
    if ((tid & 15) == 15) {
      const int rho = (tid >> 4) & 3;
#pragma unroll
      for (int i = 0; i < MB / 2; ++i) part[tid >> 6][4 * i + 2 * (rho & 1) + (rho >> 1)] = ws[i];
    }
    __syncthreads();
    if (tid < 2 * MB && mb + (tid >> 1) < m_end)
      out_rows[(mb + (tid >> 1)) * 2 + (tid & 1)] = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
  }
  __syncthreads();
}
#define DEC_MP 4                        // workgroups sharing the memory-readout terms of one unit
#define DEC_QM (IM_DM + DEC_MP * IM_D + 2 + DEC_MP)
// per unit, G * DEC_QM floats: phi(q) [G][128] | partial phi(q)^T M [DEC_MP][G][128] | gate [G] |
// unused [G] | partial phi(q)^2 . b [DEC_MP][G]

// The terms of the memory readout that do not depend on this step's eviction, for the G query heads
// of one unit against the memory state as it stands: phi_q = W_theta q, phi_q^T M, sum_c phi_q[c]^2
// b[c], and the gate sigmoid(w_g . q + c_g).  Workgroup mp of a unit takes rows 32 mp .. 32 mp + 31
// of the memory (its slice of phi_q, and partial sums over those rows).  k_dec_finish applies
// the rank-one update of this step to these terms instead of reading the updated state back.
// LDS of the prep roles (a struct, so that a kernel that also holds split workgroups can overlay it)
struct DecPrepSmem {
  float phq[DEC_GMAX][32];
  float red[4][DEC_GMAX][IM_D];
  double part[4][16];
  double rows[64 * 2];   // up to 64 batch rows x 2 outputs
  float k[IM_D];
  double u[IM_DI];
  int mp[4];
};

// Workgroups go to the 8 XCDs round-robin by their index.  Everything a unit owns (its memory state,
// readout terms, split partials, appended rows) is touched by several launches per step; with the
// unit's workgroups of every launch on XCD u % 8 those lines are found in that XCD's L2.  For a block
// range that starts at a multiple of 8 and holds `per` workgroups for each of U units (U a multiple of
// 8), index r maps to unit (r % 8) + 8 ((r / 8) / per) and item (r / 8) % per; else plain division.
__device__ __forceinline__ void xcd_unit_map(const int r, const int per, const int U, int& u, int& item) {
  if (U % 8 == 0) {
    const int x = r & 7, k = r >> 3;
    u = x + 8 * (k / per);
    item = k % per;
  } else {
    u = r / per;
    item = r % per;
  }
}

__device__ __forceinline__ void dec_prep_memory(const DecArgs& a, const int u, const int mp, DecPrepSmem& ps) {
  float (*s_phq)[32] = ps.phq;
  float (*s_red)[DEC_GMAX][IM_D] = ps.red;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = u / a.H_kv, h = u % a.H_kv, G = a.H / a.H_kv;
  float* qm = a.qm + (size_t)u * G * DEC_QM;
  // every load first
  const int d4 = tid & 31, rg = tid >> 5;    // patch of M: rows 32 mp + 4 rg .. + 3, columns 4 d4 .. 4 d4 + 3
  const float* Mu = a.M + ((size_t)(u / a.H_set) * IM_DM + 32 * mp) * IM_D;
  float4 Mr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) Mr[i] = *(const float4*)(Mu + (rg * 4 + i) * IM_D + 4 * d4);
  const int cl = tid >> 3, pt = tid & 7;     // W_theta row 32 mp + cl, dims 16 pt .. 16 pt + 15
  const uint4 Wr0 = *(const uint4*)(a.Wt + (32 * mp + cl) * IM_D + 16 * pt);
  const uint4 Wr1 = *(const uint4*)(a.Wt + (32 * mp + cl) * IM_D + 16 * pt + 8);
  const float bc = a.bvec[(size_t)(u / a.H_set) * IM_DM + 32 * mp + (lane & 31)];
  const float g0 = bf2f(a.wg[lane]), g1 = bf2f(a.wg[lane + 64]);
  const bf16_t* qb = a.q + ((size_t)b * a.H + h * G) * IM_D;
  // (the query rows too: inside the loop over the heads each pair of loads would be a round trip of its
  // own; heads past the group repeat its last row and are not used)
  uint4 qr[DEC_GMAX][2];
#pragma unroll
  for (int j = 0; j < DEC_GMAX; ++j) {
    const bf16_t* qj = qb + min(j, G - 1) * IM_D + 16 * pt;
    qr[j][0] = *(const uint4*)qj;
    qr[j][1] = *(const uint4*)(qj + 8);
  }
  float wv[16];
  unpack8(Wr0, wv);
  unpack8(Wr1, wv + 8);
#pragma unroll
  for (int j = 0; j < DEC_GMAX; ++j) {
    if (j >= G) break;
    float qv[16];
    unpack8(qr[j][0], qv);
    unpack8(qr[j][1], qv + 8);
    float pq = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) pq = fmaf(wv[e], qv[e], pq);
    // the 8 parts of a row sit in adjacent lanes: after three shifted adds lane pt = 7 has the sum
    pq += dpp_zero_f<0x111, 0xF>(pq);
    pq += dpp_zero_f<0x112, 0xF>(pq);
    pq += dpp_zero_f<0x114, 0xF>(pq);
    if (pt == 7) {
      s_phq[j][cl] = pq;
      qm[j * IM_DM + 32 * mp + cl] = pq;
    }
  }
  if (mp == 0) {
    for (int j = w; j < G; j += 4) {   // gate: one wave per head
      const float gz = wave_sum_f(fmaf(g0, bf2f(qb[j * IM_D + lane]), g1 * bf2f(qb[j * IM_D + lane + 64])));
      if (lane == 0) qm[G * (IM_DM + DEC_MP * IM_D) + j] = 1.f / (1.f + __expf(-(gz + a.cg)));
    }
  }
  __syncthreads();
  for (int j = 0; j < G; ++j) {   // partial phi_q^T M over this thread's 4 rows, then over the wave's 8
    float r0 = 0.f, r1 = 0.f, r2 = 0.f, r3 = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f = s_phq[j][rg * 4 + i];
      r0 = fmaf(f, Mr[i].x, r0); r1 = fmaf(f, Mr[i].y, r1);
      r2 = fmaf(f, Mr[i].z, r2); r3 = fmaf(f, Mr[i].w, r3);
    }
    r0 = halves_sum_f(r0); r1 = halves_sum_f(r1); r2 = halves_sum_f(r2); r3 = halves_sum_f(r3);
    if (lane < 32) *(float4*)&s_red[w][j][4 * d4] = make_float4(r0, r1, r2, r3);
  }
  for (int j = w; j < G; j += 4) {
    const float p = s_phq[j][lane & 31];
    const float dn = wave_sum_f((lane < 32) ? p * p * bc : 0.f);
    if (lane == 0) qm[G * (IM_DM + DEC_MP * IM_D + 2) + mp * G + j] = dn;
  }
  __syncthreads();
  for (int idx = tid; idx < G * IM_D; idx += 256) {
    const int j = idx >> 7, d = idx & 127;
    qm[G * IM_DM + (mp * G + j) * IM_D + d] = s_red[0][j][d] + s_red[1][j][d] + s_red[2][j][d] + s_red[3][j][d];
  }
}

// The new token of a unit: (k, v, pos) go to slot len; per-unit layout: the slot's indexer key bf16(Norm(U_k k)) is
// computed (fp64) and stored, too (head-shared layout: k_dec_finish makes it of U_k x and stores it where the token ends up).
// The set's newest position, for the recent window, and its counter for k_dec_finish are left in the workspace.
__device__ __forceinline__ void dec_prep_unit(const DecArgs& a, const int u, DecPrepSmem& ps) {
  float* s_k = ps.k;
  double* s_u = ps.u;
  int* s_mp = ps.mp;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = u / a.H_kv, su = u / a.H_set;
  const bool lead = u % a.H_set == 0;
  const int n_old = a.len[su];
  // loads that do not depend on the length go out together with it
  uint4 ukr[4], newrow;
  {
    if (!a.hs) {
      const uint4* ur = (const uint4*)(a.Uk + (tid >> 2) * IM_D + (tid & 3) * 32);
#pragma unroll
      for (int i = 0; i < 4; ++i) ukr[i] = ur[i];
    }
    // (no branch around this load: a value defined in one arm of a branch is waited for at the arm's end;
    // threads past 31 repeat thread 31's piece)
    const int t = min(tid, 31);
    newrow = *(const uint4*)(((t < 16) ? a.k_new : a.v_new) + (size_t)u * IM_D + (t & 15) * 8);
  }
  const int newpos = a.pos_new[b];
  if (lead && tid == 0) a.arrived[DEC_LINE * su] = 0;
  if (a.n_recent > 0 && a.score && lead) {  // newest position of the set (new token included) for the recent window
    int m = INT_MIN;
    const int nn = min(n_old, a.max_live);
    for (int i = tid; i < nn; i += 256) m = max(m, a.pos[(size_t)su * a.C + i]);
    if (n_old + 1 <= a.C) m = max(m, newpos);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (lane == 0) s_mp[w] = m;
    __syncthreads();
    if (tid == 0) a.maxpos[su] = max(max(s_mp[0], s_mp[1]), max(s_mp[2], s_mp[3]));
  }
  if (n_old + 1 > a.C) {
    if (tid == 0 && lead) atomicOr(a.status, IM_STATUS_APPEND_OVERFLOW_BIT);
    return;
  }
  if (n_old + 1 > a.max_live && tid == 0 && lead) atomicOr(a.status, IM_STATUS_LIVE_EXCEEDED_BIT);
  const size_t slot = (size_t)u * a.C + n_old;
  if (tid < 16) {
    *(uint4*)(a.K + slot * IM_D + tid * 8) = newrow;
    float f[8];
    unpack8(newrow, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) s_k[tid * 8 + e] = f[e];
  } else if (tid < 32) {
    *(uint4*)(a.V + slot * IM_D + (tid - 16) * 8) = newrow;
  } else if (tid == 32 && lead) {
    a.pos[(size_t)su * a.C + n_old] = newpos;
  }
  if (a.hs) return;
  __syncthreads();
  {  // u_c = Uk[c] . k : thread (c = tid/4, quarter = tid%4)
    const int c = tid >> 2, qd = tid & 3;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float f[8];
      unpack8(ukr[i], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fma((double)f[e], (double)s_k[qd * 32 + i * 8 + e], acc);
    }
    acc += __shfl_xor(acc, 1, 64);
    acc += __shfl_xor(acc, 2, 64);
    if (qd == 0) s_u[c] = acc;
  }
  __syncthreads();
  if (tid < 64) {
    const double v = s_u[tid];
    const double ss = wave_sum_d(v * v);
    const double rr = sqrt(ss / (double)IM_DI + (double)a.rms_eps);
    const double wt = a.nkw ? (double)bf2f(a.nkw[tid]) : 1.0;
    a.Kidx[slot * IM_DI + tid] = d2bf_rne(v / rr * wt);
  }
}

// projection block g: two weight rows against PR batch rows (raw projections in fp64; the consumer normalises and
// scales: it needs a whole head, this block has two of its rows)
template <int PR>
__device__ __forceinline__ void dec_prep_project(const DecArgs& a, const int g, DecPrepSmem& ps) {
  const int nB = (a.B + PR - 1) / PR;
  int rp = (nB == 1) ? g : g / nB;   // (no division on the common path)
  const int m0 = (g - rp * nB) * PR, m1 = min(m0 + PR, a.B);
  const int Nq = a.H_idx * a.di, nU = a.score ? Nq / 2 : 0, nG = a.score ? (a.H_idx + 1) / 2 : 0;
  const bool isq = rp < nU, isg = !isq && rp < nU + nG;
  const int n0 = (isq ? rp : isg ? rp - nU : rp - nU - nG) * 2;
  const int N = isq ? Nq : isg ? a.H_idx : IM_DI_SHARED;
  const bf16_t* A = isq ? a.q : a.xg;
  const bf16_t* W = isq ? a.Uq : isg ? a.Gw : a.Uk;
  const int Kd = isq ? a.H * IM_D : a.gate_in;
  double* out = isq ? a.qy : isg ? a.alpha : a.xk;
  dec_gemv2<PR>(A, W, n0, N, a.B, Kd, ps.part, ps.rows, m0, m1);
  for (int i = 2 * m0 + (int)threadIdx.x; i < 2 * m1; i += 256) {
    const int r = n0 + (i & 1);
    if (r < N) out[(size_t)(i >> 1) * N + r] = ps.rows[i];
  }
}

// --------------------------------------------------------------------------------------------
// Split workgroups
// --------------------------------------------------------------------------------------------
struct DecSplitSmem {
  float oacc[4][DEC_GMAX * IM_D];  // output partials of the 4 waves
  float wm[4][8], wl[4][8];
};

// live entries of a unit as its workgroups treat it, the new token included: at most max_live (n), and the true length
__device__ __forceinline__ int dec_true_len(int C, int n_old) { return n_old + ((n_old + 1 <= C) ? 1 : 0); }

// What the first loads of a workgroup need, as leading arguments of their own.  The build has leading arguments put into registers before a
// wave starts, which a struct never is, so the length is on its way while the rest (DecArgs) is read: one round trip of a chain of
// four (arguments, length, rows, result).  4 x 2048 entries x 8 heads, 32 layer-steps: 747 us with all in the struct, 738 with these
// arguments read from memory, 722 now; 127 steps without scores and one with, in two layers: 4160, 3976, 3893.
#define DEC_HEAD \
  const int32_t *len, const bf16_t *K, const int C, const int max_live, const int H_kv, const uint32_t kv_magic, const int H_set
struct DecHead {
  const int32_t* len;
  const bf16_t* K;
  int C, max_live, H_kv;
  uint32_t kv_magic;
  int H_set;
};

// One (unit, split) workgroup: the attention partial of its 128 keys.  The splits cover slots [0, n - 1): the last live
// one, as a rule the new token, which this launch appends, is k_dec_finish's.
__device__ __forceinline__ void dec_split(const DecArgs& a, const DecHead& hd, const int u, const int s, DecSplitSmem& sm) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // a scalar, so that branches on it are uniform
  const int b = hd.H_kv == 1 ? u : (int)__umulhi((unsigned)u, hd.kv_magic), h = u - b * hd.H_kv;   // u / H_kv, u % H_kv
  const int n = min(dec_true_len(hd.C, hd.len[hd.H_set == 1 ? u : b]), hd.max_live);
  const int k0 = s * DEC_KEYS;
  const int nk = min(DEC_KEYS, n - 1 - k0);
  if (nk <= 0) return;
  const size_t base = (size_t)u * hd.C + k0;
  const int l16 = lane & 15, kq = lane >> 4;
  // rows past the end of the split are read from its last row instead (finite values, no branches):
  // their logits are masked and their probabilities are zero further down
  uint4 kf[2][4], vf[2][4], qf[4];
  float sreg[2][4];
  // Three groups of loads per lane (K, Q, V), paced by one wait behind Q: with every workgroup of the launch resident at once,
  // issuing all 20 at the start oversubscribes the memory queues where a launch has many splits
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const int kr = min(16 * (2 * w + tt) + l16, nk - 1);
#pragma unroll
    for (int c = 0; c < 4; ++c) kf[tt][c] = load_stream16(hd.K + (base + kr) * IM_D + 32 * c + 8 * kq);
  }
  const int G = a.G;
  {
    // lanes past the group repeat its last head (their logits and probabilities are not used)
    const int jq = min(l16, G - 1);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      qf[c] = *(const uint4*)(a.q + ((size_t)b * a.H + h * G + jq) * IM_D + 32 * c + 8 * kq);
    dec_pace4();
  }
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int vr = min(16 * (2 * w + tt) + 4 * kq + i, nk - 1);
      vf[tt][i] = load_stream16(a.V + (base + vr) * IM_D + 8 * l16);
    }
  }
  // keep every load above this line, in this order: loads return in order, so each phase below
  // waits only for what it uses while the rest is still streaming in
  __asm__ volatile("" ::: "memory");
  // ---- logits of the wave's 2 tiles (bf16 MFMA, fp32 sums), softmax statistics and probabilities relative to the
  // maximum of the wave's 32 keys (the reduction below rescales), P V
  float lmax = -INFINITY;
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const im_c4 acc = att_logits(kf[tt], qf);
#pragma unroll
    for (int r = 0; r < 4; ++r) {   // this lane: head l16, key 16 (2 w + tt) + 4 kq + r
      sreg[tt][r] = (16 * (2 * w + tt) + 4 * kq + r >= nk) ? -INFINITY : acc[r] * a.scale;
      lmax = fmaxf(lmax, sreg[tt][r]);
    }
  }
  lmax = rows_max_f(lmax);               // over the wave's 32 keys, per head (lane column)
  const float mw = (lmax == -INFINITY) ? -1e30f : lmax;
  float lsum = 0.f;
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sreg[tt][r] = __expf(sreg[tt][r] - mw);   // (exp(-inf) = 0)
      lsum += sreg[tt][r];
    }
  lsum = rows_sum_f(lsum);
  if (kq == 0 && l16 < 8) { sm.wm[w][l16] = mw; sm.wl[w][l16] = lsum; }
  im_c4 o[8];
  att_pv(sreg, vf, o);
  att_store(o, sm.oacc[w], l16, kq, G);
  // the 4 waves meet in LDS
  const size_t rec = ((size_t)u * a.S + s) * G;
  __syncthreads();
  for (int idx = tid; idx < G * IM_D; idx += 256) {
    const int j = idx >> 7, d = idx & 127;
    // every wave's partial is relative to its own maximum: rescale to the split's
    const float m = fmaxf(fmaxf(sm.wm[0][j], sm.wm[1][j]), fmaxf(sm.wm[2][j], sm.wm[3][j]));
    float ov = 0.f, l = 0.f;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) {
      const float sc = __expf(sm.wm[wv][j] - m);
      ov = fmaf(sc, sm.oacc[wv][idx], ov);
      l = fmaf(sc, sm.wl[wv][j], l);
    }
    a.part[(rec + j) * IM_D + d] = ov;
    if (d == 0) a.part_ml[rec + j] = make_float2(m, l);
  }
}

// The split workgroup at index blk: consecutive ones take different units, the short last splits come last
__device__ __forceinline__ void dec_split_block(const DecArgs& a, const DecHead& hd, const int blk, const int U, DecSplitSmem& sm) {
  dec_split(a, hd, blk % U, blk / U, sm);
}

// role block r: units, then DEC_MP per unit, then projections
template <int PR>
__device__ __forceinline__ void dec_role(const DecArgs& a, const int r, DecPrepSmem& ps) {
  const int U = a.B * a.H_kv;
  if (r < U) {
    dec_prep_unit(a, r, ps);
  } else if (r < (1 + DEC_MP) * U) {
    int mu, mp;
    xcd_unit_map(r - U, DEC_MP, U, mu, mp);   // (these blocks start at grid index U: a multiple of 8 with U)
    dec_prep_memory(a, mu, mp, ps);
  } else if (r - (1 + DEC_MP) * U < a.n_proj) {
    dec_prep_project<PR>(a, r - (1 + DEC_MP) * U, ps);
  }
}

// grid: the role blocks
template <int PR>
__global__ __launch_bounds__(256) void k_dec_prep(const DecArgs a) {
  __shared__ __attribute__((aligned(16))) DecPrepSmem ps;
  dec_role<PR>(a, blockIdx.x, ps);
}

// grid: n_roles role blocks (idle ones up to a multiple of 8), then units * S split workgroups
__global__ __launch_bounds__(256, 4) void k_dec_attend(DEC_HEAD, const int n_roles, const int U, const DecArgs a) {
  __shared__ __attribute__((aligned(16))) union SM { DecSplitSmem sm; DecPrepSmem ps; __device__ SM() {} } s;
  if ((int)blockIdx.x >= n_roles) dec_split_block(a, DecHead{len, K, C, max_live, H_kv, kv_magic, H_set}, blockIdx.x - n_roles, U, s.sm);
  else dec_role<4>(a, blockIdx.x, s.ps);   // (nothing to project but U_k)
}

// --------------------------------------------------------------------------------------------
// k_dec_score
// --------------------------------------------------------------------------------------------
// the new token's indexer key in the head-shared layout, Norm(U_k x), by 16 lanes of a row (lane = dim)
__device__ __forceinline__ bf16_t dec_new_key(const DecArgs& a, const int b, const int d) {
  const double v = a.xk[(size_t)b * IM_DI_SHARED + d];
  const double ss = row16_sum_d(v * v);
  const double rr = sqrt(ss / (double)IM_DI_SHARED + (double)a.rms_eps);
  const double wk = a.nkw ? (double)bf2f(a.nkw[d]) : 1.0;
  return d2bf_rne(v / rr * wk);
}

template <int DI>
struct DecScoreSmem {
  float q[16][DI + 4];   // normalised features
  float al[16];          // gates
  bf16_t kn[16];         // head-shared layout: the new token's key
};

// A scoring workgroup (part `part` of a set's keys): 4 waves of T tiles of 16 keys.  Scores on the fp64 matrix cores, in their 4x4x4
// form: four blocks of 4 heads x 4 keys x 4 dims an instruction (16 cycles), so that 8 heads waste no columns (4 tiles: 1.75 us, 2.2
// in the 16x16x4 form, whose columns they half fill); HG groups of 4 heads, at most two at a time where a wave has several tiles: the kernel
// also streams the cache, and with all of 4 groups (184 to 210 registers) half as many workgroups fit a CU: 4 x 2048 entries, 64 query heads 30.9 us a
// layer-step with four at a time, 28.4 with two; 40 query heads 27.2, 24.8; 16 x 512, 40 heads 36.4, 34.2.  The wave's entry ranked last by (score, then position,
// then slot), with sinks and the recent window forced to the top, goes to the workspace, and the scores to the caller, if wanted.
// Bound by its chain (arguments, features, norm, products, rank): 7 us alone, hidden beside the split workgroups (10.8 us alone).
template <int DI, int T, int HG>
__device__ __forceinline__ void dec_score_block(const DecArgs& a, const int su, const int part, DecScoreSmem<DI>& sm) {
  constexpr int NH = DI == 64 ? 4 : 1, DPL = DI / 4;   // heads per wave (DI = 16: per row of 16 lanes); dims per lane of an operand
  constexpr int GP = T == 1 ? HG : 2;                  // head groups per pass over the keys (which stay in registers)
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = DI == 16 || a.H_kv == 1 ? su : (int)__umulhi((unsigned)su, a.kv_magic);
  const int group = part * 4 + w, key0 = group * 16 * T, last_row = min(a.max_live, a.C) - 1;
  // ---- raw features: head w + 4 i (tid >> 4), lane = dim
  const int d = DI == 64 ? lane : (tid & 15), j0 = DI == 64 ? w : tid >> 4;
  double yraw[NH];
#pragma unroll
  for (int i = 0; i < NH; ++i) yraw[i] = a.qy[((size_t)b * a.H_idx + min(j0 + 4 * i, a.H_idx - 1)) * DI + d];
  const double araw = a.alpha[(size_t)b * a.H_idx + min(l16, a.H_idx - 1)];
  const bf16_t wq = a.nqw ? a.nqw[d] : (bf16_t)0x3f80;
  // (in this order: the arithmetic on the features waits for them alone)
  __asm__ volatile("" ::: "memory");
  uint4 kf[T][2];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const bf16_t* row = a.Kidx + ((size_t)su * a.C + min(key0 + 16 * t + l16, last_row)) * DI;
    if constexpr (DI == 64) {
      kf[t][0] = *(const uint4*)(row + 16 * kq);
      kf[t][1] = *(const uint4*)(row + 16 * kq + 8);
    } else {
      *(uint2*)&kf[t][0] = *(const uint2*)(row + 4 * kq);
    }
  }
  // this lane ranks key l16 of tile kq (T < 4: lanes past the tiles rank nothing)
  const int own = key0 + 16 * kq + l16;
  int p = a.pos[(size_t)su * a.C + min(own, last_row)];
  const int n_old = a.len[su], qpos = a.q_pos[b], mxp = (a.n_recent > 0) ? a.maxpos[su] : 0;
  const int newpos = DI == 16 ? a.pos_new[b] : 0;
  __asm__ volatile("" ::: "memory");   // these loads go out before the arithmetic below
  if (DI == 16 && tid < 16) sm.kn[tid] = dec_new_key(a, su, tid);
  if (w == 3 && lane < 16) sm.al[lane] = lane < a.H_idx ? (float)(araw / a.alpha_denom) : 0.f;
  // ---- QK-Norm
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const int j = j0 + 4 * i;
    float f = 0.f;
    if (DI == 16 || j < a.H_idx) {   // (uniform; absent heads: zeros)
      const double ss = DI == 64 ? wave_sum_d(yraw[i] * yraw[i]) : row16_sum_d(yraw[i] * yraw[i]);
      const double rr = sqrt(ss / (double)DI + (double)a.rms_eps);
      f = j < a.H_idx ? (float)(yraw[i] / rr * (double)bf2f(wq)) : 0.f;
    }
    sm.q[j][d] = f;
  }
  // (only LDS is shared here: the keys stay in flight)
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const int n = min(dec_true_len(a.C, n_old), a.max_live);
  const int n_tiles = (n - key0 + 15) / 16;   // (of the wave that hold live keys; may be <= 0)
  float sc = 0.f;
  if (n_tiles > 0) {
    if constexpr (DI == 16) {
#pragma unroll
      for (int t = 0; t < T; ++t)
        if (key0 + 16 * t + l16 == n_old) *(uint2*)&kf[t][0] = *(const uint2*)(sm.kn + 4 * kq);
    }
    double sum[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = 0.0;
#pragma unroll 1
    for (int g0 = 0; g0 < HG; g0 += GP) {   // GP head groups at a time
      if constexpr (HG > GP) {   // (else the keys' conversions to fp64, 2 registers a value, move in front of the loop)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int i = 0; i < DPL / 8; ++i) asm volatile("" : "+v"(kf[t][i].x), "+v"(kf[t][i].y), "+v"(kf[t][i].z), "+v"(kf[t][i].w));
      }
      // left operand of head group g: lane (i = l16 % 4, kq) supplies dims DPL kq .. of head 4 g + i, alike in the 4 blocks
      float qf[GP][DPL];
#pragma unroll
      for (int g = 0; g < GP; ++g)
#pragma unroll
        for (int m = 0; m < DPL; m += 4) *(float4*)&qf[g][m] = *(const float4*)&sm.q[4 * (g0 + g) + (l16 & 3)][DPL * kq + m];
      double z[T][GP];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int g = 0; g < GP; ++g) z[t][g] = 0.0;
      auto tiles = [&](auto first, auto last) {   // tiles [first, last) together: independent chains of products
#pragma unroll
        for (int m = 0; m < DPL; ++m) {
#pragma unroll
          for (int t = first; t < last; ++t) {
            const uint4& u = kf[t][m >> 3];
            const uint32_t wd = ((m >> 1) & 3) == 0 ? u.x : ((m >> 1) & 3) == 1 ? u.y : ((m >> 1) & 3) == 2 ? u.z : u.w;
            const double k = (double)((m & 1) ? bf_hi(wd) : bf_lo(wd));
#pragma unroll
            for (int g = 0; g < GP; ++g) z[t][g] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)qf[g][m], k, z[t][g], 0, 0, 0);
          }
        }
      };
      if (T == 1 || n_tiles == 1) tiles(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
      else tiles(std::integral_constant<int, 0>{}, std::integral_constant<int, T>{});
      // result: lane (l16, kq) holds head 4 g + kq, key l16
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int g = 0; g < GP; ++g) sum[t] = fma((double)sm.al[4 * (g0 + g) + kq], fmax(z[t][g], 0.0), sum[t]);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const double all = rows_sum_d(sum[t]);
      sc = kq == t ? (float)all : sc;
    }
  }
  if (DI == 16 && own == n_old) p = newpos;
  if (p > qpos) sc = -INFINITY;   // not visible to the query
  const bool live = kq < T && own < n;
  if (a.scores && live) a.scores[(size_t)su * a.C + own] = sc;
  bool forced = p < a.n_sink;
  if (a.n_recent > 0) forced = forced || (long long)p > (long long)mxp - a.n_recent;
  const uint32_t khi = !live ? 0xffffffffu : forced ? IM_KEY_PINF : score_key(sc);
  const uint32_t klo = !live ? 0xffffffffu : (uint32_t)(~((uint32_t)p ^ 0x80000000u));
  const uint32_t mh = wave_min_u(khi);
  const uint32_t ml = wave_min_u(khi == mh ? klo : 0xffffffffu);
  const int win = (int)wave_max_u((live && khi == mh && klo == ml) ? (uint32_t)own + 1u : 0u) - 1;
  if (lane == 0 && group < a.n_pick) a.pick[(size_t)su * a.n_pick + group] = make_uint4(mh, ml, (uint32_t)win, 0u);
}

// grid: sets * ceil(n_pick / 4) scoring workgroups, idle ones up to a multiple of 8 (n_score in all), then units * S split workgroups
template <int DI, int T, int HG>
__global__ __launch_bounds__(256, 4) void k_dec_score(DEC_HEAD, const int n_score, const int U, const DecArgs a) {
  __shared__ __attribute__((aligned(16))) union SM { DecSplitSmem sm; DecScoreSmem<DI> sc; __device__ SM() {} } s;
  if ((int)blockIdx.x >= n_score) {
    dec_split_block(a, DecHead{len, K, C, max_live, H_kv, kv_magic, H_set}, blockIdx.x - n_score, U, s.sm);
    return;
  }
  const int sets = DI == 16 ? a.B : U, part = blockIdx.x / sets;
  if (4 * part < a.n_pick) dec_score_block<DI, T, HG>(a, blockIdx.x - part * sets, part, s.sc);
}

// --------------------------------------------------------------------------------------------
// k_dec_finish
// --------------------------------------------------------------------------------------------
#define DEC_FT 1024    // threads of k_dec_finish: 16 waves

template <int HPW, int DI>
struct DecFinishSmem {
  float mrg[HPW][16][IM_D];   // numerators: the waves' shares of the splits
  float phe[IM_DM];                  // phi_e
  float vrow[DI == 16 ? 16 : 1][IM_D];                  // head-shared layout: the evicted entry's V rows of the set's heads
  dec_u4 moved[DI == 16 ? 8 : 1][64];                   // head-shared layout: the last live entry's rows, pieces of 16 bytes
  bf16_t kn[16];                                        // head-shared layout: the new token's indexer key
  float xl[HPW], xe[HPW];            // logits of the last live entry and of the evicted one (behind what is read 16 bytes at a time)
  int e;                             // the evicted slot
};

// grid: (X, ceil(G / HPW), units / X), a workgroup per (unit, group of HPW query heads); X = 8 puts unit u on XCD u % 8, whose L2
// has seen its partials and readout terms.  Nobody waits for another: what they read of the cache and one of them has to
// change (the hole, the length) is changed by the last to arrive at a counter, when all have read it.  The counter needs no release and
// no acquire: every wave waits for its loads and the workgroup for its waves before it counts, so what the counter orders is reads that are
// over before one writer, and nothing that a workgroup has written is read by another in this launch.
// Bound by its chain: length, partials and ranked entries, the evicted rows, the sums (5.8 us at 4 x 2048 entries x 8 heads, 5.6 with
// the logits' digits left to chance; the form that staged a record per split took 6.1 behind a launch of 13.6 instead of 11.3).
template <int HPW, int DI>
__global__ __launch_bounds__(DEC_FT) void k_dec_finish(DEC_HEAD, const DecArgs a) {
  __shared__ __attribute__((aligned(16))) DecFinishSmem<HPW, DI> sm;
  const int G = a.G, g = blockIdx.y, u = blockIdx.x + gridDim.x * blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = H_kv == 1 ? u : (int)__umulhi((unsigned)u, kv_magic), h = u - b * H_kv;   // u / H_kv, u % H_kv
  const int su = DI == 16 ? b : u;
  const int members = (DI == 16 ? a.H_kv : 1) * gridDim.y, member = (DI == 16 ? h * gridDim.y : 0) + g;   // of the set's workgroups
  const int n_old = len[su];
  const int n_true = dec_true_len(C, n_old), n = min(n_true, max_live);   // n >= 1
  const bool over = n_true > n;   // the live-length promise is broken (flagged): nothing is evicted, the true length stays
  const int n_act = (n - 1 + DEC_KEYS - 1) / DEC_KEYS;   // splits with live keys
  const bf16_t* Ku = K + (size_t)u * C * IM_D;
  const bf16_t* Vu = a.V + (size_t)u * a.C * IM_D;
  const bf16_t* qg = a.q + ((size_t)b * a.H + h * G + g * HPW) * IM_D;   // the workgroup's first head
  const int heads = min(HPW, G - g * HPW);
  const int d = 64 * (w & 1) + lane, jw = w >> 1;   // output thread: head jw of the workgroup's, dim d
  const bool out_wave = jw < heads;
  if (DI == 16 && tid < 16) sm.kn[tid] = dec_new_key(a, su, tid);
  // ---- loads of the later phases, behind the key loads where there are any
  const int d4 = tid & 31, rg = tid >> 5;
  const int m_rows = (IM_DM + members - 1) / members, m0 = member * m_rows, m1 = min(IM_DM, m0 + m_rows);   // the workgroup's rows of M
  float* Mu = a.M + (size_t)su * IM_DM * IM_D;
  im_c4 Mr[4];
  uint4 Wr[4];                               // waves 8 - 15: rows 16 (w - 8) + l16 of W_theta; wave 5: query head l16; dims 32 c + 8 kq ..
  float b_old;
  const float* qm = a.qm + (size_t)u * G * DEC_QM;
  // (no initial values, no arithmetic on what is loaded in a branch: either makes the wave wait at the branch's end)
  float rp[DEC_MP], gate, dn;                // output waves
  bf16_t v_last, v_e;
  float2 dq;
  float m_all = -1e30f, l_all = 0.f;
  uint32_t kl_w, q_w;
  constexpr int XW = HPW <= 4 ? 4 : 8;       // waves XW .. take the last live entry's logits
  constexpr int RT = 3;                      // tiles of 16 keys in flight where a split is taken again (4: scratch)
  constexpr int PRE = HPW == 1 ? 2 : 1;   // splits per wave and head whose numerators are loaded ahead
  float2 ml[HPW], po[HPW][PRE];              // (lane = split); the wave's splits, dims 2 lane, 2 lane + 1
  constexpr int NMV = DI == 16 ? 8 : 1;
  dec_u4 mv, mvk;                            // wave 7: the last live entry's rows (they move into the hole; head-shared: in LDS)
  int mvpos;
  const float* pu = a.part + (size_t)u * a.S * G * IM_D;   // (offsets of 64 bits: a unit's partials exceed 2^31 floats from 2^28 entries on)
  const float2* mlu = a.part_ml + (size_t)u * a.S * G;
  auto merge_loads = [&]() {
#pragma unroll
    for (int jj = 0; jj < HPW; ++jj) {
      const int j = g * HPW + min(jj, heads - 1);
      ml[jj] = mlu[min(lane, a.S - 1) * G + j];
#pragma unroll
      for (int k = 0; k < PRE; ++k)
        if (w + 16 * k < n_act) po[jj][k] = *(const float2*)(pu + (size_t)((w + 16 * k) * G + j) * IM_D + 2 * lane);
    }
  };
  auto wave_loads = [&]() {   // what a wave has to do behind the decision
    if (w >= 8) {
#pragma unroll
      for (int c = 0; c < 4; ++c) Wr[c] = *(const uint4*)(a.Wt + (16 * (w - 8) + l16) * IM_D + 32 * c + 8 * kq);
    }
    if (w == 5) {
#pragma unroll
      for (int c = 0; c < 4; ++c) Wr[c] = *(const uint4*)(qg + min(l16, heads - 1) * IM_D + 32 * c + 8 * kq);
    }
    if (w >= XW && w < XW + heads) {   // the last live entry's logits: a wave per head
      kl_w = *(const uint32_t*)(Ku + (size_t)(n - 1) * IM_D + 2 * lane);
      q_w = *(const uint32_t*)(qg + (w - XW) * IM_D + 2 * lane);
    }
    if (out_wave) {
      const int j = g * HPW + jw;
#pragma unroll
      for (int k = 0; k < DEC_MP; ++k) rp[k] = qm[G * IM_DM + (k * G + j) * IM_D + d];
      gate = qm[G * (IM_DM + DEC_MP * IM_D) + j];
      dq = *(const float2*)(qm + j * IM_DM + 2 * lane);
      dn = qm[G * (IM_DM + DEC_MP * IM_D + 2) + min(lane, DEC_MP - 1) * G + j];
      v_last = Vu[(size_t)(n - 1) * IM_D + d];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (32 * i < m_rows) Mr[i] = *(const im_c4*)(Mu + min(m0 + rg + 32 * i, m1 - 1) * IM_D + 4 * d4);   // (rows past m1: not used)
    if (member == 0 && (w == 2 || w == 3)) b_old = a.bvec[(size_t)su * IM_DM + d];
    if (w == 7) {
#pragma unroll
      for (int i = 0; i < NMV; ++i) {   // pieces of 16 bytes: head (lane >> 5) + 2 i, K then V
        if (2 * i >= a.H_set) break;    // (uniform)
        const int hm = min((lane >> 5) + 2 * i, a.H_set - 1), pc = lane & 31;
        const bf16_t* src = ((pc < 16) ? a.K : a.V) + (((size_t)su * a.H_set + hm) * a.C + (n - 1)) * IM_D + (pc & 15) * 8;
        if constexpr (DI == 16) copy_to_lds_1k((const char*)src, (char*)sm.moved[i]);
        else mv = *(const dec_u4*)src;
      }
      mvk = *(const dec_u4*)(a.Kidx + ((size_t)su * a.C + (n - 1)) * DI + min(lane, DI / 8 - 1) * 8);
      mvpos = a.pos[(size_t)su * a.C + (n - 1)];
    }
  };
  // numerators relative to the maximum over all splits, which every wave finds for itself
  auto head_max = [&](int jj) {
    float m = lane < n_act ? ml[jj].x : -1e30f;
    for (int sp = lane + 64; sp < n_act; sp += 64) m = fmaxf(m, mlu[sp * G + g * HPW + jj].x);
    return wave_max_f(m);
  };
  auto merge = [&]() {
#pragma unroll
    for (int jj = 0; jj < HPW; ++jj) {
      const bool mine = out_wave && jj == jw;
      if (jj >= heads || (w >= n_act && !mine)) continue;   // (uniform)
      const float m = head_max(jj);
      if (mine) {
        m_all = m;
        l_all = lane < n_act ? ml[jj].y * __expf(ml[jj].x - m) : 0.f;
        for (int sp = lane + 64; sp < n_act; sp += 64) {
          const float2 t = mlu[sp * G + g * HPW + jj];
          l_all = fmaf(t.y, __expf(t.x - m), l_all);
        }
        l_all = wave_sum_f(l_all);
        dn = wave_sum_f(lane < DEC_MP ? dn : 0.f);
      }
      float o0 = 0.f, o1 = 0.f;
#pragma unroll
      for (int k = 0; k < PRE; ++k) {
        if (w + 16 * k < n_act) {
          const float sc = __expf(readlane_f(ml[jj].x, w + 16 * k) - m);   // (a split below 64)
          o0 = fmaf(sc, po[jj][k].x, o0);
          o1 = fmaf(sc, po[jj][k].y, o1);
        }
      }
      for (int sp = w + 16 * PRE; sp < n_act; sp += 16) {
        const int at = sp * G + g * HPW + jj;
        const float sc = __expf(mlu[at].x - m);
        const float2 v = *(const float2*)(pu + (size_t)at * IM_D + 2 * lane);
        o0 = fmaf(sc, v.x, o0);
        o1 = fmaf(sc, v.y, o1);
      }
      *(float2*)&sm.mrg[jj][w][2 * lane] = make_float2(o0, o1);
    }
    if (w >= XW && w < XW + heads) {
      const float xl = wave_sum_f(fmaf(bf_lo(kl_w), bf_lo(q_w), bf_hi(kl_w) * bf_hi(q_w))) * a.scale;
      if (lane == 0) sm.xl[w - XW] = xl;
    }
  };
  // ---- the evicted slot: one wave takes the last-ranked entry of all while the others' loads go out (a wave that does both
  // waits for all it has loaded, since part of it is loaded in branches)
  int e = -1;
  const bool decide = a.n_pick > 0 && n > a.budget && !over;
  if (decide) {
    if (w == 6) {
      const uint4* pick = a.pick + (size_t)su * a.n_pick;
      uint4 r = pick[min(lane, a.n_pick - 1)];   // (an entry that is looked at twice changes nothing)
      const uint4 r2 = pick[min(lane + 64, a.n_pick - 1)];
      // (groups ascend: on a full tie the later one has the larger slot)
      auto later = [&](const uint4& x) {
        if ((int)x.z >= 0 && ((int)r.z < 0 || x.x < r.x || (x.x == r.x && x.y <= r.y))) r = x;
      };
      later(r2);
      for (int i = lane + 128; i - lane < a.n_pick; i += 256) {   // (four at a time: a load that is waited for by itself is a round trip)
        uint4 x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = pick[min(i + 64 * k, a.n_pick - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) later(x[k]);
      }
      const bool on = (int)r.z >= 0;
      const uint32_t khi = on ? r.x : 0xffffffffu, klo = on ? r.y : 0xffffffffu;
      const uint32_t mh = wave_min_u(khi);
      const uint32_t mlo = wave_min_u(khi == mh ? klo : 0xffffffffu);
      const int s = (int)wave_max_u((on && khi == mh && klo == mlo) ? r.z + 1u : 0u) - 1;
      if (lane == 0) sm.e = s;
    }
  } else if (a.named) {
    e = a.named[su];
  }
  merge_loads();
  wave_loads();
  if (decide) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (the loads stay in flight)
    e = sm.e;
  } else {
    e = (e >= 0 && e < n && !over) ? e : -1;
  }
  e = __builtin_amdgcn_readfirstlane(e);
  // ---- the evicted entry's rows
  uint4 ke[4];
  uint2 ve_w;
  if (e >= 0) {
    const bf16_t* Ke = Ku + (size_t)e * IM_D;
    const bf16_t* Ve = Vu + (size_t)e * IM_D;
    if (w == 5 || w >= 8) {   // (the memory takes the rows summed over the set's heads: column l16 of the product below is head l16's)
      const bf16_t* kr = DI == 64 || w == 5 ? Ke : a.K + (((size_t)su * a.H_kv + min(l16, a.H_kv - 1)) * a.C + e) * IM_D;
#pragma unroll
      for (int c = 0; c < 4; ++c) ke[c] = *(const uint4*)(kr + 32 * c + 8 * kq);
    }
    if (DI == 16) {
      if (w < 8) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int hm = w + 8 * i;
          if (hm < a.H_kv) {
            const uint32_t x = *(const uint32_t*)(a.V + (((size_t)su * a.H_kv + hm) * a.C + e) * IM_D + 2 * lane);
            *(float2*)&sm.vrow[hm][2 * lane] = make_float2(bf_lo(x), bf_hi(x));
          }
        }
      }
    } else {
      ve_w = *(const uint2*)(Ve + 4 * d4);
    }
    if (out_wave) v_e = Ve[d];
  }
  merge();
  // The evicted entry's logits by the product that its split has used, operands on the same sides: the same bits, so that what is
  // subtracted below is what its partial holds, however large the logits are (another order of the 128 terms: off by up to 1e-4 at 300)
  if (w == 5 && e >= 0) {
    const im_c4 z = att_logits(ke, Wr);
    if (kq == 0 && l16 < heads) sm.xe[l16] = z[0] * a.scale;
  }
  // ---- phi_e = W_theta k_e on the matrix cores: waves 8 - 15 take 16 rows each.  Every column of the product is k_e; head-shared
  // layout: column l16 is head l16's key, and the columns are added.  Products are exact, and the four parts of a sum are added as a tree:
  // a chain through the accumulator has 6.0e-8 of the sum as its error, the tree 4.8e-8, 128 terms on the vector ALU 5.1e-8.
  if (e >= 0 && w >= 8) {
    im_c4 part[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      part[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(im_bf8, Wr[c]), __builtin_bit_cast(im_bf8, ke[c]),
                                                       im_c4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    im_c4 z = (part[0] + part[1]) + (part[2] + part[3]);
    if constexpr (DI == 16) {
#pragma unroll
      for (int r = 0; r < 4; ++r) z[r] = row16_sum_f(l16 < a.H_kv ? z[r] : 0.f);
    }
    if (l16 == 0) *(float4*)&sm.phe[16 * (w - 8) + 4 * kq] = make_float4(z[0], z[1], z[2], z[3]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's reads of the cache have returned ...
  __syncthreads();                                    // ... and those of the whole workgroup
  int arrived = 0;
  if (w == 7 && lane == 0) arrived = __hip_atomic_fetch_add(a.arrived + DEC_LINE * su, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // ---- output of (head jw, dim d)
  if (out_wave) {
    const int j = g * HPW + jw;
    // the splits' maximum and denominator, the waves' shares, the last live entry, less the evicted one
    float m = m_all, l = l_all, o = 0.f;
    const float xl = sm.xl[jw], xe = sm.xe[jw], share_e = sm.mrg[jw][(max(e, 0) / DEC_KEYS) & 15][d];   // (on their way beside the shares)
    float sizes = 0.f;   // of the shares
    auto shares = [&](auto count) {   // (all reads first: one latency instead of one for every four)
      float x[count];
#pragma unroll
      for (int i = 0; i < count; ++i) x[i] = sm.mrg[jw][i][d];
#pragma unroll
      for (int i = 0; i < count; ++i) {
        const float y = i < n_act ? x[i] : 0.f;   // (the others hold nothing)
        o += y;
        sizes += fabsf(y);
      }
    };
    if (n_act > 4) shares(std::integral_constant<int, 16>{});
    else shares(std::integral_constant<int, 4>{});
    const float ve_last = bf2f(v_last), ve_d = e >= 0 ? bf2f(v_e) : 0.f;
    // phi_q . phi_e, the readout's denominator, and
    // phi_q^T (lambda M + eta phi_e v_e^T) = lambda phi_q^T M + eta (phi_q . phi_e) v_e.  (Without a branch around it, and before the
    // branch below: a chain beside the other)
    float mr = (rp[0] + rp[1]) + (rp[2] + rp[3]);
    static_assert(DEC_MP == 4, "four parts of phi_q^T M");
    const float2 pp = *(const float2*)&sm.phe[2 * lane];
    const float dt = wave_sum_f(fmaf(dq.x, pp.x, dq.y * pp.y));
    const float sq = wave_sum_f(fmaf(dq.x * dq.x, pp.x * pp.x, dq.y * dq.y * pp.y * pp.y));
    float v_sum = ve_d;
    if constexpr (DI == 16) {
      v_sum = 0.f;
      for (int i = 0; i < a.H_kv; ++i) v_sum += sm.vrow[i][d];
    }
    dn = e >= 0 ? fmaf(a.lambda, dn, a.eta * sq) : dn;
    mr = e >= 0 ? fmaf(a.lambda, mr, a.eta * dt * v_sum) : mr;
    const float res = gate * (mr / (dn + a.mem_eps));
    auto add = [&](float m2, float l2, float o2) {
      const float mn = fmaxf(m, m2), s1 = __expf(m - mn), s2 = __expf(m2 - mn);
      o = fmaf(o, s1, s2 * o2);
      l = fmaf(l, s1, s2 * l2);
      m = mn;
    };
    if (e != n - 1) {
      add(xl, 1.f, ve_last);
      if (e >= 0) {
        // The evicted entry is in its split's partial, and its share of the sums has their rounding errors.  They are subtracted
        // where that leaves enough of the sums: 1 / 16 of the denominator (the errors count 16 times: 1e-6 of the output, whose half step is 2e-3),
        // and in this dim 1 / 256 of the evicted entry's part (by chance or design a dim may have next to nothing else: 2e-5 of it), more of it
        // the further its logit lies below the maximum: an exponent of size D is rounded by 2^-24 D, so the errors grow as 4 + D and the line
        // goes down with them (D = 25 with 1 / 256: 4e-4 of the dim).  What stays
        // is at least the sum of the sizes of the waves' shares without it.  Else (or with an infinity or NaN in sight) its split is taken again
        // without it, which costs the launch 5 us (13 with a row a lane): with lines of 1 / 2 and 1 / 16 that is every launch where a few keys
        // dominate (16 x 512 entries, one key in 20 four times as long: 891 us a pass, 776 now).
        const float pe = __expf(xe - m), pv = pe * ve_d, l0 = l;
        const float to_m = __expf(m_all - m);
        const float stays = fmaf(to_m, sizes - fabsf(share_e), fabsf(fmaf(to_m, share_e, -pv)) + fabsf(__expf(xl - m) * ve_last));
        l -= pe;
        o -= pv;
        if (__builtin_expect(__any(!(pe <= 0.9375f * l0) || !(fabsf(pv) * (4.f + (m - xe)) <= 1024.f * stays) || !(stays < 1e37f)), 0)) {
          // (the hole may be filled meanwhile: its row is not read).  The wave's shares have been read; its half of their rows is scratch now
          const int se = e / DEC_KEYS, k0 = se * DEC_KEYS, nk = min(DEC_KEYS, n - 1 - k0);
          float (*tmp)[IM_D] = (float (*)[IM_D])&sm.mrg[jw][0][64 * (w & 1)];   // [16][64], rows IM_D apart
          auto in = [&](int key) { return key < nk && k0 + key != e; };
          auto row = [&](int key) { return in(key) ? k0 + key : n - 1; };   // (others: the last live entry's, not added)
          {
            uint4 qf[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) qf[c] = *(const uint4*)(qg + jw * IM_D + 32 * c + 8 * kq);
#pragma unroll 1
            for (int t0 = 0; 16 * t0 < nk; t0 += RT) {   // (every load of RT tiles, then the products; all columns are the head)
              uint4 kf[RT][4];
#pragma unroll
              for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int c = 0; c < 4; ++c) kf[t][c] = *(const uint4*)(Ku + (size_t)row(16 * (t0 + t) + l16) * IM_D + 32 * c + 8 * kq);
#pragma unroll
              for (int t = 0; t < RT; ++t) {
                const im_c4 z = att_logits(kf[t], qf);
                const int key = 16 * (t0 + t) + 4 * kq;
                if (l16 == 0) *(float4*)&tmp[key >> 6][key & 63] = make_float4(z[0], z[1], z[2], z[3]);
              }
            }
          }
          float lg[2], p2[2];
#pragma unroll
          for (int x = 0; x < 2; ++x) {   // lane: keys lane, lane + 64
            const int key = lane + 64 * x;
            lg[x] = in(key) ? tmp[x][lane] * a.scale : -INFINITY;
          }
          m = fmaxf(wave_max_f(fmaxf(lg[0], lg[1])), -1e30f);
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            p2[x] = __expf(lg[x] - m);
            tmp[x][lane] = p2[x];
          }
          l = wave_sum_f(p2[0] + p2[1]);
          {
            const int rw = lane >> 3, dc = 8 * (lane & 7);   // 8 rows of 64 dims a load
            float acc[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll 1
            for (int k = 0; k < nk; k += 64) {
              uint4 vr[8];
#pragma unroll
              for (int i = 0; i < 8; ++i) vr[i] = *(const uint4*)(Vu + (size_t)row(k + 8 * i + rw) * IM_D + 64 * (w & 1) + dc);
#pragma unroll
              for (int i = 0; i < 8; ++i) {
                const int key = k + 8 * i + rw;
                const float pr = tmp[key >> 6][key & 63];
                float v[8];
                unpack8(vr[i], v);
                if (in(key)) {
#pragma unroll
                  for (int c = 0; c < 8; ++c) acc[c] = fmaf(pr, v[c], acc[c]);
                }
              }
            }
            *(float4*)&tmp[2 + rw][dc] = make_float4(acc[0], acc[1], acc[2], acc[3]);
            *(float4*)&tmp[2 + rw][dc + 4] = make_float4(acc[4], acc[5], acc[6], acc[7]);
            o = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) o += tmp[2 + i][lane];
          }
#pragma unroll 1
          for (int sp = 0; sp < n_act; sp += 8) {
            float2 r[8];
            float ov[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int at = min(sp + i, n_act - 1) * G + j;
              r[i] = mlu[at];
              ov[i] = pu[(size_t)at * IM_D + d];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
              if (sp + i < n_act && sp + i != se) add(r[i].x, r[i].y, ov[i]);
          }
          add(xl, 1.f, ve_last);
        }
      }
    }
    const float o_attn = (l > 0.f) ? o / l : 0.f;
    const size_t oi = ((size_t)b * a.H + h * G + j) * IM_D + d;
    a.out[oi] = f2bf_rne(o_attn + res);
    if (a.readout) a.readout[oi] = res;
  }
  if (e >= 0) {
    // M <- lambda M + eta phi_e v_e^T for this thread's rows, 4 columns each; b <- lambda b + eta phi_e^2
    float4 ve4;
    if constexpr (DI == 16) {
      ve4 = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m0 + rg < m1) {
        for (int i = 0; i < a.H_kv; ++i) {
          const float4 v = *(const float4*)&sm.vrow[i][4 * d4];
          ve4.x += v.x; ve4.y += v.y; ve4.z += v.z; ve4.w += v.w;
        }
      }
    } else {
      ve4 = make_float4(bf_lo(ve_w.x), bf_hi(ve_w.x), bf_lo(ve_w.y), bf_hi(ve_w.y));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + rg + 32 * i;
      if (row < m1) {
        const float f = a.eta * sm.phe[row];
        const im_c4 m = Mr[i];
        *(float4*)(Mu + row * IM_D + 4 * d4) =
            make_float4(fmaf(a.lambda, m[0], f * ve4.x), fmaf(a.lambda, m[1], f * ve4.y), fmaf(a.lambda, m[2], f * ve4.z),
                        fmaf(a.lambda, m[3], f * ve4.w));
      }
    }
    if (member == 0 && (w == 2 || w == 3)) {
      const float pe = sm.phe[d];
      a.bvec[(size_t)su * IM_DM + d] = fmaf(a.lambda, b_old, a.eta * pe * pe);
    }
  }
  // ---- every workgroup of the set has read the cache: the last live entry into the hole, the new length
  if (w != 7 || __builtin_amdgcn_readfirstlane(arrived) != members - 1) return;
  const int n_keep = (e >= 0) ? n - 1 : n;
  const bool new_key = DI == 16 && n_old + 1 <= a.C;   // head-shared layout: the new token's key is not in the cache yet
  if (e >= 0 && e < n_keep) {
#pragma unroll
    for (int i = 0; i < NMV; ++i) {
      const int hm = (lane >> 5) + 2 * i, pc = lane & 31;
      if (hm < a.H_set)
        *(dec_u4*)(((pc < 16) ? a.K : a.V) + (((size_t)su * a.H_set + hm) * a.C + e) * IM_D + (pc & 15) * 8) = DI == 16 ? sm.moved[i][lane] : mv;
    }
    if (lane < DI / 8 && !new_key) *(dec_u4*)(a.Kidx + ((size_t)su * a.C + e) * DI + lane * 8) = mvk;
    if (lane == 0) a.pos[(size_t)su * a.C + e] = mvpos;
  }
  if (new_key && lane < IM_DI_SHARED) {
    // the new token sits in the last live slot, unless that entry has just moved into the hole (or is the evicted one)
    const int at = (e >= 0 && e < n_keep) ? e : n_true - 1;
    if (e != n - 1) a.Kidx[((size_t)su * a.C + at) * IM_DI_SHARED + lane] = sm.kn[lane];
  }
  if (lane == 0) {
    a.len[su] = over ? n_true : n_keep;
    a.nproj[su] = over ? n_true : n_keep;
    if (a.evicted) a.evicted[su] = e;
    if (a.score && n > a.budget + 1) atomicOr(a.status, IM_STATUS_OVER_BUDGET_BIT);
  }
}
