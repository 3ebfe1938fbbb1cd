// Large products of bf16 matrices with an exact sum: C[m][n] = sum_k A[m][k] B[n][k], rounded to fp64 once.
//
// The query projection of a prompt needs fp64 sums of 4096 bf16 products (everything that decides an eviction
// is taken in fp64), and the fp64 matrix cores give 78 TFLOP/s.  The int8 ones give 5000: a row is written as
// integers of a common unit, x = X 2^(E - 149) with E the row's largest (biased) exponent, so |X| <= 255 2^22, in four
// signed base-256 digits, and the 16 products of digits, accumulated exactly in 7 int32 sums (one per power of
// 256), give the exact sum of X W: a third of the time of the fp64 cores.  Elements more than 2^22 below their
// row's largest lose bits in X: a row lists up to XG_ROOM of them (1 in 2.6 million values, for Gaussian ones), and their
// remainders' products are added in fp64 afterwards, in a fixed order.  So an element of C is the exact sum rounded
// once, where neither its row nor its column lists anything; else, one fp64 sum of the remainders is added to that.
// A row with more of them, an infinity or a NaN is full: the 64 x 64 tiles of C that it is part of are computed
// on the fp64 cores instead.
// Every row writes its count and its exponent anew: nothing is kept from one product to the next.
//   k_exact_prep : row exponents and lists; digit planes of B
//   k_exact_gemm : the product
//   k_exact_fix  : remainders
#pragma once
#include "im_kernels.h"

typedef int im_i4 __attribute__((ext_vector_type(4)));
typedef int im_i16 __attribute__((ext_vector_type(16)));

#define XG_BM 64            // rows of A, rows of B, and contraction length per workgroup step
#define XG_BN 128
#define XG_BK 64
#define XG_MAX_K 8192       // sums of 4 digit products stay below 2^29, and the two halves of the result below 2^53
#define XG_ROOM 8           // listed elements of a row
#define XG_FULL (XG_ROOM + 1)
// Rows of A, then of B: the number of listed elements (or XG_FULL), and their k, ascending.
struct ExactLists {
  int32_t *countA, *countB;
  uint16_t *a, *b;   // [row][XG_ROOM]
};

// the scale 2^(149 - E) that makes a row's elements integers; rows of very small numbers take a larger unit
__device__ __forceinline__ int exact_clamp_exp(int e) { return max(e, 40); }
__device__ __forceinline__ float exact_scale(int e) { return __uint_as_float((uint32_t)(127 + 156 - e) << 23); }
// (unit of X: 2^(E - 127 - 7 - 22) = 2^(E - 156))

// the largest exponent of 8 bf16 values
__device__ __forceinline__ int exact_max_exp(const uint4& u, int e) {
  const uint32_t v[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) e = max(e, (int)max((v[i] >> 7) & 255u, (v[i] >> 23) & 255u));
  return e;
}

// which of 8 values X truncates
__device__ __forceinline__ uint32_t exact_lost(const uint4& u, float scale) {
  const uint32_t v[4] = {u.x, u.y, u.z, u.w};
  uint32_t lost = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float f = ((i & 1) ? bf_hi(v[i >> 1]) : bf_lo(v[i >> 1])) * scale;
    lost |= (f != truncf(f)) ? 1u << i : 0u;
  }
  return lost;
}

// 8 values -> their 4 digit planes (8 bytes each, lowest digit first)
__device__ __forceinline__ void exact_digits(const uint4& u, float scale, uint2 (&plane)[4]) {
  const uint32_t v[4] = {u.x, u.y, u.z, u.w};
  uint32_t x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int xi = (int)(((i & 1) ? bf_hi(v[i >> 1]) : bf_lo(v[i >> 1])) * scale);   // towards zero
    // digits d_0 .. d_3 in -128 .. 127: the bytes of X + 0x80808080, each less 128
    x[i] = ((uint32_t)xi + 0x80808080u) ^ 0x80808080u;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {                    // 4 x 4 byte transpose
    const uint32_t a = x[4 * h], b = x[4 * h + 1], c = x[4 * h + 2], d = x[4 * h + 3];
    const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    const uint32_t p0 = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u), p1 = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    const uint32_t p2 = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u), p3 = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
    if (h == 0) { plane[0].x = p0; plane[1].x = p1; plane[2].x = p2; plane[3].x = p3; }
    else { plane[0].y = p0; plane[1].y = p1; plane[2].y = p2; plane[3].y = p3; }
  }
}

// x - X unit for a listed element
__device__ __forceinline__ double exact_rest(bf16_t x, int e) {
  const float f = bf2f(x) * exact_scale(e);
  return ldexp((double)f - (double)(int)f, e - 156);
}

// Byte offset, inside the operand of a 32-row tile and a 32-wide step, of digit plane 0 of 8 values k = 8 p .. (p = 0 .. 3)
// of a row: lane (row % 32, k / 16) of the 32x32x32 product reads 16 bytes.  A plane has 1 KB.
__device__ __forceinline__ int exact_place(int row, int p) { return (((p >> 1) * 32 + (row & 31)) << 4) + (p & 1) * 8; }

// grid (ceil(M / 4) + ceil(Np / 4)), one wave per row; Np = N rounded up to XG_BN (rows past N are zeros).
// expA [M], expB [Np]; planes [Np / 32][K / 32][4 digits][1 KB]
__global__ __launch_bounds__(256) void k_exact_prep(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, int M, int N,
                                                    int Np, int K, int32_t* __restrict__ expA,
                                                    int32_t* __restrict__ expB, char* __restrict__ planes,
                                                    ExactLists lists) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, mb = (M + 3) / 4;
  const bool isb = (int)blockIdx.x >= mb;
  const int row = (isb ? (int)blockIdx.x - mb : (int)blockIdx.x) * 4 + w;
  if (row >= (isb ? Np : M)) return;
  const bf16_t* src = isb ? B + (size_t)min(row, N - 1) * K : A + (size_t)row * K;
  uint4 v[XG_MAX_K / 512];   // the row: 8 values per lane and piece (absent pieces repeat the first)
  const int pieces = K / 512, rest = K % 512;
#pragma unroll
  for (int i = 0; i < XG_MAX_K / 512; ++i) {
    if (i * 512 < K) v[i] = *(const uint4*)(src + ((i < pieces || lane * 8 < rest) ? i * 512 + lane * 8 : 0));
  }
  int e = 0;
#pragma unroll
  for (int i = 0; i < XG_MAX_K / 512; ++i)
    if (i * 512 < K) e = exact_max_exp(v[i], e);
  e = exact_clamp_exp((int)wave_max_u((uint32_t)e));
  if (lane == 0) (isb ? expB : expA)[row] = e;
  const float scale = row < N || !isb ? exact_scale(e) : 0.f;
  unsigned long long lost[2] = {0ull, 0ull};   // of this lane's values: 8 bits per piece
#pragma unroll
  for (int i = 0; i < XG_MAX_K / 512; ++i) {
    const int k = i * 512 + lane * 8;
    if (i * 512 >= K || k >= K) continue;
    lost[i / 8] |= (unsigned long long)exact_lost(v[i], scale) << (8 * (i % 8));
    if (!isb) continue;
    uint2 pl[4];
    exact_digits(v[i], scale, pl);
    char* dst = planes + ((size_t)(row / 32) * (K / 32) + k / 32) * 4096 + exact_place(row, (k / 8) & 3);
#pragma unroll
    for (int d = 0; d < 4; ++d) *(uint2*)(dst + d * 1024) = pl[d];
  }
  int count = e == 255 ? XG_FULL : 0;
  if (__any((lost[0] | lost[1]) != 0ull)) {   // (in practice a handful of rows in the whole matrix)
    uint16_t* list = (isb ? lists.b : lists.a) + (size_t)row * XG_ROOM;
    for (int i = 0; i * 512 < K && count < XG_FULL; ++i) {
      const uint32_t bits = (uint32_t)((i < 8 ? lost[0] : lost[1]) >> (8 * (i & 7))) & 255u;
      unsigned long long lanes = __ballot(bits != 0u);
      while (lanes && count < XG_FULL) {
        const int ln = __builtin_ctzll(lanes);
        lanes &= lanes - 1;
        uint32_t of = (uint32_t)__builtin_amdgcn_readlane((int)bits, ln);
        while (of && count < XG_FULL) {
          if (count < XG_ROOM && lane == 0) list[count] = (uint16_t)(i * 512 + ln * 8 + __builtin_ctz(of));
          of &= of - 1;
          ++count;
        }
      }
    }
  }
  if (lane == 0) (isb ? lists.countB : lists.countA)[row] = count;
}

// grid (ceil(M / XG_BM) * Np / XG_BN), 8 waves as 2 x 4; a wave owns a 32 x 32 tile of C in 7 int32 accumulators.
// A step is 64 values of the contraction: 32 products of 32 cycles per wave, two waves per SIMD, 0.85 us.  B's planes are
// copied straight into LDS and A's rows (bf16) too, three steps ahead (a load from HBM takes up to 2 us); the thread
// that copied 8 values of A turns them into digits one step ahead, between the products.  A step has two halves of 16
// products; the operands of a half are read from LDS during the half before it (read at the top of a step, by all
// waves at once, they took 1024 cycles of the LDS in which no product ran), so the step's barrier lies between
// its halves.  65536 x 512 x 4096: 1563 us (1737 with the operands read at the top of a step and 8 rows per wave's copy); the
// clock is 2.04 GHz under it.  fp64 matrix cores: 4441 us.
__global__ __launch_bounds__(512, 2) void k_exact_gemm(const bf16_t* __restrict__ A, const char* __restrict__ planes,
                                                       const int32_t* __restrict__ expA,
                                                       const int32_t* __restrict__ expB, double* __restrict__ C, int M,
                                                       int N, int Np, int K) {
  __shared__ __attribute__((aligned(16))) char sA[2][XG_BM * XG_BK * 4], sB[3][XG_BN * XG_BK * 4];
  __shared__ __attribute__((aligned(16))) char sR[3][XG_BM * XG_BK * 2];   // A's rows as they are
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w & 1, wn = w >> 1;
  // workgroups go to the 8 XCDs round-robin: an XCD keeps to one column tile where there are 1, 2, 4 or 8 of them, so
  // that its part of B's planes stays in its L2
  const int nt = Np / XG_BN, bid = blockIdx.x;
  int tn, tm;
  if (8 % nt == 0) { tn = (bid & 7) % nt; tm = (bid >> 3) * (8 / nt) + (bid & 7) / nt; }
  else { tn = bid % nt; tm = bid / nt; }
  const int m0 = tm * XG_BM, n0 = tn * XG_BN;
  if (m0 >= M) return;
  // this thread's piece of A: row arow, values 8 ap .. of every step (a wave has 32 rows of 32 bytes: the digits of 8 rows of
  // 128 bytes met in the same banks four at a time)
  const int arow = (w >> 2) * 32 + (lane >> 1), ap = 2 * (w & 3) + (lane & 1);
  const int am = min(m0 + arow, M - 1);
  const bf16_t* asrc = A + (size_t)am * K + ap * 8;
  const int nc = K / XG_BK;
  const float ascale = exact_scale(expA[am]);
  const int aplace = ((arow >> 5) * 2 + (ap >> 2)) * 4096 + exact_place(arow, ap & 3);
  // a step's copies: 8 KB of A (each wave what its threads convert), 4 row tiles x 2 steps x 4 KB of B
  auto fetchA = [&](int c, int buf) { copy_to_lds_1k((const char*)(asrc + min(c, nc - 1) * XG_BK), &sR[buf][w * 1024]); };
  auto fetchB = [&](int c, int buf) {
    c = min(c, nc - 1);   // (past the end: not used)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int piece = w * 4 + i, t = piece >> 3, rest = piece & 7;
      copy_to_lds_1k(planes + ((size_t)(n0 / 32 + t) * (K / 32) + 2 * c) * 4096 + rest * 1024 + lane * 16, &sB[buf][piece * 1024]);
    }
  };
  im_i16 acc[7];
#pragma unroll
  for (int p = 0; p < 7; ++p)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[p][r] = 0;
  auto digits = [&](int raw, int buf) {   // this thread's values: digit planes into LDS
    uint2 pl[4];
    exact_digits(*(const uint4*)(&sR[raw][tid * 16]), ascale, pl);
#pragma unroll
    for (int d = 0; d < 4; ++d) *(uint2*)(&sA[buf][aplace + d * 1024]) = pl[d];
  };
  auto operands = [&](im_i4* a, im_i4* b, int bufA, int bufB, int st) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      a[d] = *(const im_i4*)(&sA[bufA][(wm * 2 + st) * 4096 + d * 1024 + lane * 16]);
      b[d] = *(const im_i4*)(&sB[bufB][(wn * 2 + st) * 4096 + d * 1024 + lane * 16]);
    }
  };
  // pairs of digits in an order that leaves other sums between two products of the same sum
  auto products = [&](const im_i4* a, const im_i4* b) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int j = (d + s) & 3;
        acc[d + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[d], b[j], acc[d + j], 0, 0, 0);
      }
  };
  fetchA(0, 0);
  fetchA(1, 1);
  fetchB(0, 0);
  fetchA(2, 2);
  fetchB(1, 1);
  copy_wait<5>();
  digits(0, 0);
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the raw values have been read
  fetchA(3, 0);
  fetchB(2, 2);
  __syncthreads();
  im_i4 a0[4], b0[4], a1[4], b1[4];
  operands(a0, b0, 0, 0, 0);
  int bA = 0, b3 = 0;
#pragma unroll 1
  for (int c = 0; c < nc; ++c) {
    const int next = b3 == 2 ? 0 : b3 + 1;
    // first half; the second half's operands and the next step's digits on their way
    operands(a1, b1, bA, b3, 1);
    digits(next, bA ^ 1);
    products(a0, b0);
    // (a product keeps the matrix core busy for 8 vector instructions)
    __builtin_amdgcn_sched_group_barrier(0x100, 9, 0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x200, 4, 0);
    copy_wait<5>();    // all but the youngest group of copies: B of the next step and A of the one after it are here
    __syncthreads();   // ... for every wave; this step's operands and the next step's raw values have been read
    fetchA(c + 4, next);
    fetchB(c + 3, b3);
    operands(a0, b0, bA ^ 1, next, 0);
    products(a1, b1);
    bA ^= 1;
    b3 = next;
  }
  copy_wait<0>();
  // result register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
  const int n = n0 + 32 * wn + (lane & 31);
  if (n >= N) return;
  const int eb = expB[n];
  int4 ea[4];   // (rows past M: words of the workspace behind the exponents, not used)
#pragma unroll
  for (int i = 0; i < 4; ++i) ea[i] = *(const int4*)(expA + m0 + 32 * wm + 8 * i + 4 * (lane >> 5));
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + 32 * wm + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int em = (r & 3) == 0 ? ea[r >> 2].x : (r & 3) == 1 ? ea[r >> 2].y : (r & 3) == 2 ? ea[r >> 2].z : ea[r >> 2].w;
    if (m >= M) continue;
    // both parts are exact (|acc| <= 2^29): one rounding
    const double lo = fma(fma(fma((double)acc[3][r], 256.0, (double)acc[2][r]), 256.0, (double)acc[1][r]), 256.0, (double)acc[0][r]);
    const double hi = fma(fma((double)acc[6][r], 256.0, (double)acc[5][r]), 256.0, (double)acc[4][r]);
    C[(size_t)m * N + n] = ldexp(fma(hi, 4294967296.0, lo), em + eb - 312);
  }
}

// remainders of an element of C, a row of A (its listed k, their number, the values, the exponent) and one of B: those of a
// against the whole of b, then those of b against the integers of a, each in ascending order of k
__device__ __forceinline__ double exact_remainder(const uint4& la, int ca, const bf16_t* ar, int ea, const uint4& lb, int cb,
                                                  const bf16_t* br, int eb) {
  const uint32_t a[4] = {la.x, la.y, la.z, la.w}, b[4] = {lb.x, lb.y, lb.z, lb.w};
  double sum = 0.0;
#pragma unroll
  for (int j = 0; j < XG_ROOM; ++j) {
    if (j < ca) {
      const int k = (a[j / 2] >> (16 * (j & 1))) & 0xffffu;
      sum = fma(exact_rest(ar[k], ea), (double)bf2f(br[k]), sum);
    }
  }
#pragma unroll
  for (int j = 0; j < XG_ROOM; ++j) {
    if (j < cb) {
      const int k = (b[j / 2] >> (16 * (j & 1))) & 0xffffu;
      sum = fma(exact_rest(br[k], eb), (double)bf2f(ar[k]) - exact_rest(ar[k], ea), sum);
    }
  }
  return sum;
}

// remainders: grid (ceil(N / 64) * ceil(M / 64)), a workgroup per 64 x 64 tile of C, which returns at once where nothing is
// listed.  Its waves take the listed rows of A in turn (lane = column), then the listed columns (lane = row, of the rows
// that list nothing): an element has one owner.  A chain of three loads per row; with a thread per element, which met its
// listed ones one after another, a prompt of 2 x 1500 tokens with one value listed in B took 12 us longer.
__global__ __launch_bounds__(256) void k_exact_fix(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, int M, int N, int K,
                                                   const int32_t* __restrict__ expA, const int32_t* __restrict__ expB,
                                                   double* __restrict__ C, ExactLists lists) {
  const int tx = (N + 63) / 64, bx = blockIdx.x % tx, by = blockIdx.x / tx, m0 = by * 64, n0 = bx * 64;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ca = (m0 + lane < M) ? lists.countA[m0 + lane] : 0, cb = (n0 + lane < N) ? lists.countB[n0 + lane] : 0;
  if (!__any(ca | cb)) return;   // (every wave looks at all 128 counts)
  if (__any(ca > XG_ROOM || cb > XG_ROOM)) {
    gemm_nt_tile<2, 2>(A, B, C, M, N, K, bx, by);
    return;
  }
  const unsigned long long rows = __ballot(ca > 0), cols = __ballot(cb > 0);
  const int ea = expA[min(m0 + lane, M - 1)], eb = expB[min(n0 + lane, N - 1)];
  int turn = 0;
  for (unsigned long long r = rows; r; r &= r - 1) {
    if ((turn++ & 3) != w) continue;
    const int i = __builtin_ctzll(r), m = m0 + i, n = min(n0 + lane, N - 1);
    const uint4 la = *(const uint4*)(lists.a + (size_t)m * XG_ROOM);
    uint4 lb = make_uint4(0, 0, 0, 0);
    if (cb > 0) lb = *(const uint4*)(lists.b + (size_t)n * XG_ROOM);
    double* c = C + (size_t)m * N + n;
    const double old = *c;
    const double sum = exact_remainder(la, __builtin_amdgcn_readlane(ca, i), A + (size_t)m * K, __builtin_amdgcn_readlane(ea, i), lb, cb,
                                       B + (size_t)n * K, eb);
    if (n0 + lane < N) *c = old + sum;
  }
  for (unsigned long long r = cols; r; r &= r - 1) {
    if ((turn++ & 3) != w) continue;
    const int i = __builtin_ctzll(r), n = n0 + i, m = min(m0 + lane, M - 1);
    const uint4 lb = *(const uint4*)(lists.b + (size_t)n * XG_ROOM);
    double* c = C + (size_t)m * N + n;
    const double old = *c;
    const double sum = exact_remainder(make_uint4(0, 0, 0, 0), 0, A + (size_t)m * K, ea, lb, __builtin_amdgcn_readlane(cb, i), B + (size_t)n * K,
                                       __builtin_amdgcn_readlane(eb, i));
    if (m0 + lane < M && ca == 0) *c = old + sum;
  }
}
