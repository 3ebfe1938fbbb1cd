// libindexmem: host side of the C ABI declared in include/indexmem.h.
// Validation happens first and touches no GPU; the rest only enqueues kernels on the caller's
// stream.  No device memory is allocated here.
#include "../../include/indexmem.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "im_kernels.h"
#include "im_score.h"
#include "im_exact.h"
#include "im_decode.h"

struct im_handle {
  im_config cfg;
  char* ws;
  size_t ws_bytes;
  int max_live;
  bool ws_ready;
  // workspace layout (byte offsets)
  size_t off_status, off_qy, off_alpha, off_mem, off_attn, off_dpart, off_dml, off_dqm, off_xk, off_dpick, off_darrived, total;
  size_t off_xexp, off_xcount, off_xplanes, off_xlist;              // exact products
  size_t off_spart, off_qf, off_al16, off_qblk, off_recu, off_reci, off_nlist, off_list;   // scores of several queries
  int attn_chunks;
  // optional kernel timing (im_profile_start / im_profile_stop)
  hipEvent_t* prof_ev;
  int prof_max, prof_n, prof_span;
  char err[256];
};

// Scratch of the entry point that allocates nothing (im_decode_attn_with_readout_static): a status
// word in the first 256 bytes, then the attention partials.  Every GPU the library runs on holds
// its own copy of this array, at its own address, until the process ends.  In host code the name is
// only a handle for hipGetSymbolAddress: the per-device address it returns is what kernels, fills and
// copies are given.
#define IM_STATIC_MAX_DEVICES 64
static __device__ __align__(256) unsigned char im_static_scratch[IM_STATIC_SCRATCH_BYTES];
static void* g_static_ptr[IM_STATIC_MAX_DEVICES];
static std::mutex g_static_mu;
static thread_local char g_static_err[256] = "";

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int set_err(im_handle* h, int code, const char* fmt, ...) {
  if (h) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(h->err, sizeof(h->err), fmt, ap);
    va_end(ap);
  }
  return code;
}

// the calling thread's error text of a call that takes no handle (im_last_error(NULL))
int static_err(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_static_err, sizeof(g_static_err), fmt, ap);
  va_end(ap);
  return code;
}

const char* config_problem(const im_config* c, int* code) {
  *code = IM_ERR_INVALID_ARG;
  if (!c) return "config is NULL";
  if (c->batch < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1) return "batch and head counts must be >= 1";
  if (c->n_q_heads % c->n_kv_heads != 0) return "n_q_heads must be a multiple of n_kv_heads";
  if (c->capacity < 1) return "capacity must be >= 1";
  if (c->n_idx_heads < 1 || c->n_idx_heads > 16) return "n_idx_heads must be in 1..16";
  if (c->gate_in_dim < 16 || c->gate_in_dim % 16 != 0) return "gate_in_dim must be a positive multiple of 16";
  if (c->n_sink < 0 || c->n_recent < 0) return "n_sink and n_recent must be >= 0";
  if ((long long)c->n_sink + c->n_recent > c->capacity) return "n_sink + n_recent exceeds capacity";
  if (c->fold_block < 32 || c->fold_block % 32 != 0) return "fold_block must be a positive multiple of 32";
  if (c->max_queries < 1) return "max_queries must be >= 1";
  if (!(c->rms_eps >= 0.f) || !(c->mem_eps > 0.f) || !(c->softmax_scale > 0.f))
    return "rms_eps >= 0, mem_eps > 0 and softmax_scale > 0 are required";
  if ((long long)c->batch * c->n_kv_heads > 65535) return "batch * n_kv_heads must be <= 65535";
  if (c->head_shared != 0 && c->head_shared != 1) return "head_shared must be 0 or 1";
  *code = IM_ERR_UNSUPPORTED;
  if (c->head_dim != IM_D) return "head_dim must be 128";
  if (c->idx_dim != (c->head_shared ? IM_DI_SHARED : IM_DI)) return "idx_dim must be 64 (16 with head_shared = 1)";
  if (c->mem_dim != IM_DM) return "mem_dim must be 128";
  if (c->n_q_heads / c->n_kv_heads > 8) return "more than 8 query heads per KV head";
  *code = IM_OK;
  return nullptr;
}

size_t score_block_bytes(const im_config* c) {
  if (c->head_shared) return c->n_idx_heads <= 8 ? ScoreBlock<IM_DI_SHARED, 8>::BYTES : ScoreBlock<IM_DI_SHARED, 16>::BYTES;
  return c->n_idx_heads <= 8 ? ScoreBlock<IM_DI, 8>::BYTES : ScoreBlock<IM_DI, 16>::BYTES;
}

// workgroups a scan aims at: with query groups it has at most this many (rounded up by one group), and a
// workgroup covers at most 256 keys, which bounds its records
#define IM_SCORE_WGS 2048
#define IM_SCORE_GROUP_TILES 512   // fewer tiles of 256 keys: a short window's queries go in groups
size_t score_rec_keys(size_t sets, size_t capacity) {
  const size_t all = IM_SCORE_GROUPS * sets * capacity, few = (size_t)IM_SCORE_WGS * 256 + sets * capacity;
  return all < few ? all : few;
}

// Up to this many keys a wave of k_score_exact takes 4 instead of 16, which it evaluates in turn.  Scoring calls of 2000 queries, 4
// keys a wave against 16, in us: 12000 keys 190 / 200, 24000 keys 207 / 213, 32768 keys 220 / 224 (head-shared 252 /
// 247), 48000 keys 267 / 262, 65536 keys 298 / 290.
#define IM_EXACT_FEW 32768
// The query projection of M rows goes through the exact int8 product (im_exact.h) where it has more than 2048 tiles
// of 16 x 16: below, its 64 x 128 tiles leave most of the chip idle and the fp64 kernel that splits the contraction is
// faster (512 rows x 512: 32 us against 80).  Up to 32 columns stay there too: the exact product has 128 of them in any case
// (scoring calls of 65536 rows x 4096, exact against fp64: 16 columns 793 / 459 us, 32 columns 752 / 618, 48
// columns 753 / 860).
size_t exact_np(const im_config* c) { return ((size_t)c->n_idx_heads * c->idx_dim + XG_BN - 1) / XG_BN * XG_BN; }
bool exact_fits(const im_config* c, long long M) {
  const long long N = c->n_idx_heads * c->idx_dim, K = (long long)c->n_q_heads * IM_D;
  return N > 32 && K <= XG_MAX_K && M < (1 << 30) && ((M + 15) / 16) * ((N + 15) / 16) > 2048;
}

size_t n_sets_of(const im_config* c) { return (size_t)c->batch * (c->head_shared ? 1 : c->n_kv_heads); }

// Splits of a set's evicted rows over workgroups (k_mem_partial*), `live` bounding their number: as many as give the 512
// workgroups that the chip holds, of at least 64 rows (sets of several heads: 1024, of 32 rows of every head; 8 sets x 3072
// rows x 8 heads: 99 us with 256 workgroups, 105 with 384, 86 with 768).  A tile of 32 rows
// takes a workgroup 5 us per head, a partial of 64 KB far less.  8 units x 1167 rows: 2 splits 79 us, 24 splits 14 us;
// 8 units x 4096 rows: 8 splits 68 us, 64 splits 23 us.
int splits_of(long long live, long long rows, long long wgs, long long sets) {
  const long long n = (live + rows - 1) / rows, most = (wgs + sets - 1) / sets;
  return (int)(n < most ? n : most);
}
int mem_splits(const im_config* c, long long live) {
  return c->head_shared ? splits_of(live, 32, 1024, n_sets_of(c)) : splits_of(live, 64, 512, n_sets_of(c));
}
// whether a call may go through the bounds: shorter windows never do (score_short)
bool score_may_scan(const im_config* c) {
  return c->max_queries > 16 && (long long)((c->max_queries + 15) / 16) * c->n_idx_heads * c->idx_dim > 512;
}

// The status words stay from call to call.  Everything else is written and read inside one call, and calls on one handle
// do not overlap: what grows with the queries comes first, and behind it scoring, memory write, attention and the
// fused steps use the same memory, one after another.
void layout(const im_config* c, im_handle* h) {
  const size_t B = c->batch, Hi = c->n_idx_heads, units = (size_t)c->batch * c->n_kv_heads, sets = n_sets_of(c);
  auto take = [](size_t& off, size_t bytes) {
    const size_t at = off;
    off = align256(off + bytes);
    return at;
  };
  size_t base = 0;
  // status word (in a 32-word slot of its own), then one newest-position word per unit
  h->off_status = take(base, (32 + units) * sizeof(int32_t));
  // raw query projections and gates (of the fused steps, too)
  const size_t rows = B * c->max_queries, qblk = (c->max_queries + 15) / 16;
  h->off_qy = take(base, rows * Hi * c->idx_dim * sizeof(double));
  h->off_alpha = take(base, rows * Hi * sizeof(double));
  // the query projection as an exact product
  const size_t np = exact_np(c), xk = (size_t)c->n_q_heads * IM_D;
  const bool exact = exact_fits(c, (long long)c->batch * c->max_queries);
  const size_t xrows = exact ? rows + np : 0;
  h->off_xexp = take(base, xrows * sizeof(int32_t));
  h->off_xcount = take(base, xrows * sizeof(int32_t));
  h->off_xlist = take(base, xrows * XG_ROOM * sizeof(uint16_t));
  h->off_xplanes = take(base, exact ? np * xk * 4 : 0);
  // scores by bounds: normalised features, gates, operand blocks of 16 queries, counts of listed keys
  const bool scan = score_may_scan(c);
  h->off_qf = take(base, scan ? rows * Hi * c->idx_dim * sizeof(float) : 0);
  h->off_al16 = take(base, scan ? rows * 16 * sizeof(float) : 0);
  h->off_qblk = take(base, scan ? B * qblk * score_block_bytes(c) : 0);
  h->off_nlist = take(base, scan ? B * sizeof(int32_t) : 0);
  size_t score = base, mem = base, attn = base, step = base;
  // ... the scan's records, listed keys
  const size_t rec_keys = scan ? score_rec_keys(sets, c->capacity) : 0;
  h->off_recu = take(score, rec_keys * 4 * sizeof(float2));
  h->off_reci = take(score, rec_keys * 4 * sizeof(int32_t));
  h->off_list = take(score, scan ? sets * c->capacity * sizeof(int2) : 0);
  // short windows: the query groups' maxima over a short cache (fewer than IM_SCORE_GROUP_TILES tiles of 256 keys)
  const size_t most = (size_t)IM_SCORE_GROUP_TILES * 256, few_keys = sets * c->capacity < most ? sets * c->capacity : most;
  h->off_spart = take(score, c->max_queries > 16 ? IM_SCORE_GROUPS * few_keys * sizeof(float) : 0);
  // memory write: partial sums (at most 34 MB, 68 MB with sets of several heads)
  h->off_mem = take(mem, sets * mem_splits(c, c->capacity) * (IM_DM * IM_D + IM_DM) * sizeof(float));
  // attention
  h->attn_chunks = (c->capacity + IM_ATT_CHUNK - 1) / IM_ATT_CHUNK;
  h->off_attn = take(attn, B * c->n_q_heads * h->attn_chunks * IM_ATT_REC * sizeof(float));
  // the fused steps; head_shared: U_k X of the rows of one append or step, fp64
  const size_t splits = (c->capacity + DEC_KEYS - 1) / DEC_KEYS, G = c->n_q_heads / c->n_kv_heads;
  h->off_dpart = take(step, units * splits * G * IM_D * sizeof(float));
  h->off_dml = take(step, units * splits * G * sizeof(float2));
  h->off_dqm = take(step, units * G * DEC_QM * sizeof(float));
  h->off_xk = take(step, c->head_shared ? B * c->capacity * IM_DI_SHARED * sizeof(double) : 0);
  h->off_dpick = take(step, sets * ((c->capacity + 15) / 16) * sizeof(uint4));
  h->off_darrived = take(step, DEC_LINE * sets * sizeof(int32_t));
  h->total = score;
  for (size_t end : {mem, attn, step}) h->total = end > h->total ? end : h->total;
}

int launch_check(im_handle* h, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_err(h, IM_ERR_LAUNCH, "%s: %s", what, hipGetErrorString(e));
  return IM_OK;
}

int ensure_ws(im_handle* h, hipStream_t s) {
  if (h->ws_ready) return IM_OK;
  const int n_words = 32 + h->cfg.batch * h->cfg.n_kv_heads;
  k_fill_i32<<<(n_words + 255) / 256, 256, 0, s>>>((int32_t*)(h->ws + h->off_status), n_words, 0);
  int rc = launch_check(h, "workspace clear");
  if (rc == IM_OK) h->ws_ready = true;
  return rc;
}

int32_t* status_ptr(im_handle* h) { return (int32_t*)(h->ws + h->off_status); }

bool state_ok(const im_state* st) {
  return st && st->K && st->V && st->Kidx && st->pos && st->len && st->n_projected && st->M && st->b;
}
bool params_ok(const im_params* p) { return p && p->Uq && p->G && p->Uk && p->Wtheta && p->wg; }

// KV heads per set, and the number of sets (what lengths, lists and the memory state are kept per)
int heads_per_set(const im_config& c) { return c.head_shared ? c.n_kv_heads : 1; }
int n_sets(const im_config& c) { return c.batch * c.n_kv_heads / heads_per_set(c); }

#define IM_REQUIRE(cond, msg) \
  do { if (!(cond)) return set_err(h, IM_ERR_INVALID_ARG, "%s: %s", __func__, msg); } while (0)

// The last launch of a fused step: a workgroup of 16 waves fills a CU, so it takes the fewest query heads with which the
// launch fits the chip once, or all of the unit's.  us per layer-step with 1, 2, 4, 8 heads, per unit: 32 units of 4 heads 21.4, 22.1, 23.9, 24.5; 64 of
// 4 23.0, 23.7, 25.6, 26.1; 64 of 7 24.9, 22.3, 23.4, 25.5; 64 of 8 35.7, 33.1, 34.6, 36.8; 128 of 8 50.7, 44.8, 43.0, 44.7; 320 of 8 88.5, 74.9, 71.7, 71.4; 512
// of 8 147, 124, 116, 111; 512 of 4 79, 70, 66, 67.  Head-shared: 32 of 8 23.2, 23.4, 25.4, 28.3; 64 of 8 28.5, 24.8, 26.5, 28.2; 128 of 8 41.1, 33.8, 30.8, 32.4;
// 320 of 8 71.6, 54.0, 48.4, 45.4; 512 of 4 81.6, 66.2, 60.5, 61.7; 512 of 8 116, 87, 75, 66.
template <int HPW, int DI>
void launch_finish_as(const DecArgs& a, hipStream_t s) {
  const int units = a.B * a.H_kv, x = units % 8 == 0 ? 8 : 1;
  k_dec_finish<HPW, DI><<<dim3(x, (a.G + HPW - 1) / HPW, units / x), DEC_FT, 0, s>>>(a.len, a.K, a.C, a.max_live, a.H_kv, a.kv_magic, a.H_set, a);
}
template <int DI>
void launch_finish(const DecArgs& a, hipStream_t s) {
  const int units = a.B * a.H_kv, G = a.G;
  if (units * G <= 256 || G == 1) launch_finish_as<1, DI>(a, s);
  else if (units * ((G + 1) / 2) <= 256 || G == 2) launch_finish_as<2, DI>(a, s);
  else if (units * ((G + 3) / 4) <= 256 || G <= 4) launch_finish_as<4, DI>(a, s);
  else launch_finish_as<8, DI>(a, s);
}

// The launches of a fused step; begin and end (events, or NULL) are recorded behind the first and behind the one that streams the cache
template <int DI, int HG>
void launch_score(const DecArgs& a, int tiles, hipStream_t s) {
  const int units = a.B * a.H_kv, sets = units / a.H_set, n_score = (sets * ((a.n_pick + 3) / 4) + 7) / 8 * 8;
  const int blocks = n_score + units * a.S;
  auto launch = [&](auto kernel) { kernel<<<blocks, 256, 0, s>>>(a.len, a.K, a.C, a.max_live, a.H_kv, a.kv_magic, a.H_set, n_score, units, a); };
  if constexpr (DI == IM_DI_SHARED || HG == 2) {
    if (tiles == 4) return launch(k_dec_score<DI, 4, HG>);
  }
  if constexpr (DI == IM_DI) {
    if (tiles == 1) return launch(k_dec_score<DI, 1, HG>);
  }
  launch(k_dec_score<DI, 2, HG>);
}
void launch_step(const DecArgs& a, int n_roles, int prep_rows, int tiles, hipEvent_t begin, hipEvent_t end, hipStream_t s) {
  const int units = a.B * a.H_kv;
  if (!a.score) {
    k_dec_attend<<<n_roles + units * a.S, 256, 0, s>>>(a.len, a.K, a.C, a.max_live, a.H_kv, a.kv_magic, a.H_set, n_roles, units, a);
  } else {
    if (prep_rows == 4) k_dec_prep<4><<<n_roles, 256, 0, s>>>(a);
    else k_dec_prep<8><<<n_roles, 256, 0, s>>>(a);
    if (begin) (void)hipEventRecord(begin, s);
    if (a.hs) {
      if (a.H_idx <= 8) launch_score<IM_DI_SHARED, 2>(a, tiles, s); else launch_score<IM_DI_SHARED, 4>(a, tiles, s);
    } else {
      if (a.H_idx <= 8) launch_score<IM_DI, 2>(a, tiles, s); else launch_score<IM_DI, 4>(a, tiles, s);
    }
  }
  if (end) (void)hipEventRecord(end, s);
  if (a.hs) launch_finish<IM_DI_SHARED>(a, s);
  else launch_finish<IM_DI>(a, s);
}

// C[m][n] = sum_k A[m][k] B[n][k] in fp64: matrix cores when the contraction length allows; the contraction
// split over 16 or 4 waves for small products (more waves, shorter chains), 2 x 2 tiles per wave for large ones
// (less L2 traffic)
long long gemm_tiles(long long M, long long N) { return ((M + 15) / 16) * ((N + 15) / 16); }
void gemm_nt(hipStream_t s, const bf16_t* A, const bf16_t* B, double* Cm, int M, int N, int Kd) {
  if (Kd % 32 != 0) {
    k_gemm_nt_f64<<<dim3((N + 63) / 64, (M + 63) / 64), 256, 0, s>>>(A, B, Cm, M, N, Kd);
  } else if (Kd % 512 == 0 && gemm_tiles(M, N) <= 512) {
    // (the gates of 4096 queries: 20 us with 4 waves a tile, 15 with 16; of 32768: 95 with 4 or 8)
    k_gemm_nt_mfma_split<16><<<dim3((M + 15) / 16, (N + 15) / 16), 1024, 0, s>>>(A, B, Cm, M, N, Kd);
  } else if (Kd % 128 == 0 && (N <= 16 || gemm_tiles(M, N) <= 2048)) {
    k_gemm_nt_mfma_split<4><<<dim3((M + 15) / 16, (N + 15) / 16), 256, 0, s>>>(A, B, Cm, M, N, Kd);
  } else if ((long long)M * N <= (1ll << 21) || N <= 16) {
    k_gemm_nt_mfma<1, 1><<<dim3((N + 31) / 32, (M + 31) / 32), 256, 0, s>>>(A, B, Cm, M, N, Kd);
  } else {
    k_gemm_nt_mfma<2, 2><<<dim3((N + 63) / 64, (M + 63) / 64), 256, 0, s>>>(A, B, Cm, M, N, Kd);
  }
}

// the query projection of M rows as an exact product (exact_fits)
void exact_project(im_handle* h, hipStream_t s, const bf16_t* q, const bf16_t* Uq, double* y, int M) {
  const im_config& c = h->cfg;
  const int N = c.n_idx_heads * c.idx_dim, K = c.n_q_heads * IM_D, np = (int)exact_np(&c);
  int32_t* expA = (int32_t*)(h->ws + h->off_xexp);
  const size_t rows = (size_t)c.batch * c.max_queries;   // (the rows of B come behind those of A)
  int32_t *expB = expA + rows, *count = (int32_t*)(h->ws + h->off_xcount);
  uint16_t* list = (uint16_t*)(h->ws + h->off_xlist);
  char* planes = h->ws + h->off_xplanes;
  const ExactLists lists = {count, count + rows, list, list + rows * XG_ROOM};
  k_exact_prep<<<(M + 3) / 4 + (np + 3) / 4, 256, 0, s>>>(q, Uq, M, N, np, K, expA, expB, planes, lists);
  const int nt = np / XG_BN, mt = (M + XG_BM - 1) / XG_BM, per = 8 % nt == 0 ? 8 / nt : 1;
  k_exact_gemm<<<(mt + per - 1) / per * per * nt, 512, 0, s>>>(q, planes, expA, expB, y, M, N, np, K);
  k_exact_fix<<<(N + 63) / 64 * ((M + 63) / 64), 256, 0, s>>>(q, Uq, M, N, K, expA, expB, y, lists);
}

// A short window of queries (n_q >= H_idx) is scored in fp64 against all keys: per key that takes, for 16 queries,
// H_idx d_idx operations, and up to 512 of them cost less than the bounds and their candidates; over a short cache, whose
// queries go in groups, more of them do.  Scoring calls, fp64 against bounds, in us:
//   16 queries x 8 heads of 64 dims: 65536 keys 49 / 73, 524288 keys 188 / 250; 24 queries 70 / 77 and 330 / 271
//   16 queries x 16 heads of 64, 131072 keys: 144 / 183; 24 queries 196 / 166
//   64 queries x 8 heads of 16, 512 keys 29 / 35, 8192 keys 31 / 37, 131072 keys 68 / 87
//   32 queries x 8 heads of 64, 4096 keys 42 / 46, 22400 keys 59 / 58; 64 queries 37 / 42 and 93 / 75
//   24 queries x 8 heads of 64: 32768 keys 51 / 56, 65536 keys 70 / 77, 96000 keys 87 / 91; 40 queries 67 / 58, 99 / 86, 126 / 101
long long score_tiles(const im_handle* h) { return (long long)((h->max_live + 255) / 256) * n_sets_of(&h->cfg); }
bool score_short(const im_handle* h, int n_q) {
  const im_config& c = h->cfg;
  const long long ops = (long long)((n_q + 15) / 16) * c.n_idx_heads * c.idx_dim, keys = (long long)h->max_live * n_sets_of(&c);
  if (!score_may_scan(&c)) return true;   // (the workspace holds nothing for the bounds)
  return n_q <= 16 || ops <= 512 || (score_tiles(h) < 128 && n_q <= 128 && ops * keys <= 24000000) ||
         (score_tiles(h) < IM_SCORE_GROUP_TILES && n_q <= 32 && ops <= 1024);
}

// the scores of longer windows from their raw projections in the workspace
template <int DI, int HM>
void score_many(im_handle* h, const im_state* st, const bf16_t* norm_q_w, const int32_t* q_pos, int n_q,
                double alpha_denom, float* scores, hipStream_t s) {
  const im_config& c = h->cfg;
  const int units = n_sets(c), per_b = units / c.batch, live = h->max_live, nblk = (n_q + 15) / 16;
  char* ws = h->ws;
  float* qf = (float*)(ws + h->off_qf);
  float* al16 = (float*)(ws + h->off_al16);
  char* blocks = ws + h->off_qblk;
  float2* rec_u = (float2*)(ws + h->off_recu);
  int32_t* rec_i = (int32_t*)(ws + h->off_reci);
  int32_t* n_listed = (int32_t*)(ws + h->off_nlist);
  int2* listed = (int2*)(ws + h->off_list);
  const bf16_t* Kidx = (const bf16_t*)st->Kidx;
  k_score_features<DI, HM><<<dim3(nblk, c.batch), 1024, 0, s>>>((const double*)(ws + h->off_qy),
      (const double*)(ws + h->off_alpha), q_pos, norm_q_w, c.rms_eps, alpha_denom, n_q, c.n_idx_heads, qf, al16, blocks,
      n_listed);
  // a scan over a short cache has few (256-key tile, unit) workgroups: its query blocks then go in up to
  // IM_SCORE_GROUPS groups with workgroups of their own; a very short one also drops to 16 keys per wave
  const long long tiles4 = (long long)((live + 255) / 256) * units;
  const bool small = tiles4 * IM_SCORE_GROUPS < 1024;
  const int tiles = small ? (live + 63) / 64 : (live + 255) / 256;
  int groups = (int)((IM_SCORE_WGS + (long long)tiles * units - 1) / ((long long)tiles * units));
  if (groups > IM_SCORE_GROUPS) groups = IM_SCORE_GROUPS;
  if (groups > nblk) groups = nblk;
  const int per_group = (nblk + groups - 1) / groups;
  groups = (nblk + per_group - 1) / per_group;
  const dim3 grid(tiles * units, groups);
  if (small)
    k_score_scan<DI, HM, 1><<<grid, 256, 0, s>>>(Kidx, st->pos, st->len, st->n_projected, blocks, q_pos, n_q, per_b,
                                                 c.capacity, c.n_idx_heads, live, units, per_group, live, rec_u, rec_i);
  else
    k_score_scan<DI, HM, 4><<<grid, 256, 0, s>>>(Kidx, st->pos, st->len, st->n_projected, blocks, q_pos, n_q, per_b,
                                                 c.capacity, c.n_idx_heads, live, units, per_group, live, rec_u, rec_i);
  // the wave's keys are evaluated in turn, 1.5 us each
  if ((long long)live * units <= IM_EXACT_FEW)
    k_score_exact<DI, HM, 4><<<dim3((live + 15) / 16, units), 256, 0, s>>>(
        Kidx, st->pos, st->len, blocks, qf, al16, q_pos, n_q, per_b, c.capacity, c.n_idx_heads, live, groups, live, rec_u,
        rec_i, scores, n_listed, listed);
  else
    k_score_exact<DI, HM, 16><<<dim3((live + 63) / 64, units), 256, 0, s>>>(
        Kidx, st->pos, st->len, blocks, qf, al16, q_pos, n_q, per_b, c.capacity, c.n_idx_heads, live, groups, live, rec_u,
        rec_i, scores, n_listed, listed);
  k_score_listed<DI, HM><<<IM_LIST_WGS, 256, 0, s>>>(Kidx, st->pos, blocks, qf, al16, c.batch, n_q, per_b, c.capacity,
                                             c.n_idx_heads, scores, n_listed, listed);
}

}  // namespace

extern "C" {

size_t im_workspace_bytes(const im_config* cfg) {
  int code;
  if (config_problem(cfg, &code)) return 0;
  im_handle tmp;
  layout(cfg, &tmp);
  return tmp.total;
}

int32_t im_create(const im_config* cfg, void* workspace, size_t workspace_bytes, im_handle** out) {
  if (!out) return IM_ERR_INVALID_ARG;
  *out = nullptr;
  int code;
  if (config_problem(cfg, &code)) return code;
  im_handle* h = (im_handle*)calloc(1, sizeof(im_handle));
  if (!h) return IM_ERR_LAUNCH;
  h->cfg = *cfg;
  layout(cfg, h);
  if (!workspace || ((uintptr_t)workspace & 255) != 0 || workspace_bytes < h->total) {
    free(h);
    return IM_ERR_INVALID_ARG;
  }
  h->ws = (char*)workspace;
  h->ws_bytes = workspace_bytes;
  h->max_live = cfg->capacity;
  h->ws_ready = false;
  h->err[0] = 0;
  *out = h;
  return IM_OK;
}

static void release_profile(im_handle* h) {
  if (!h->prof_ev) return;
  for (int i = 0; i < 2 * h->prof_max; ++i) (void)hipEventDestroy(h->prof_ev[i]);
  free(h->prof_ev);
  h->prof_ev = nullptr;
  h->prof_max = h->prof_n = 0;
}

void im_destroy(im_handle* h) {
  if (!h) return;
  release_profile(h);
  free(h);
}

int32_t im_profile_start(im_handle* h, int32_t max_records, int32_t span) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(max_records >= 1 && max_records <= (1 << 20), "max_records must be in 1..2^20");
  IM_REQUIRE(span >= IM_PROFILE_MAIN && span <= IM_PROFILE_PREP_AND_MAIN, "span must be one of IM_PROFILE_*");
  release_profile(h);
  h->prof_ev = (hipEvent_t*)calloc(2 * (size_t)max_records, sizeof(hipEvent_t));
  if (!h->prof_ev) return set_err(h, IM_ERR_LAUNCH, "im_profile_start: out of host memory");
  h->prof_max = max_records;
  for (int i = 0; i < 2 * max_records; ++i) {
    hipError_t e = hipEventCreate(&h->prof_ev[i]);
    if (e != hipSuccess) {
      h->prof_max = i / 2;
      release_profile(h);
      return set_err(h, IM_ERR_LAUNCH, "hipEventCreate: %s", hipGetErrorString(e));
    }
  }
  h->prof_n = 0;
  h->prof_span = span;
  return IM_OK;
}

int32_t im_stream_read(const void* src, size_t bytes, uint32_t never, void* sink, void* stream) {
  if (!src || !sink || bytes < 16 || bytes % 16 != 0 || ((uintptr_t)src & 15) != 0)
    return static_err(IM_ERR_INVALID_ARG, "im_stream_read: src / sink is NULL, or bytes / src is not a multiple of 16");
  // 8 workgroups of 4 waves per CU: 2048 workgroups, each thread 8 x 16 bytes per round
  k_stream_read<<<2048, 256, 0, (hipStream_t)stream>>>((const uint4*)src, bytes / 16, never, (uint32_t*)sink);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return static_err(IM_ERR_LAUNCH, "im_stream_read: %s", hipGetErrorString(e));
  return IM_OK;
}

int32_t im_profile_stop(im_handle* h, float* ms_host, int32_t* n_records, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(ms_host && n_records, "ms_host / n_records is NULL");
  IM_REQUIRE(h->prof_ev, "im_profile_start was not called");
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) return set_err(h, IM_ERR_LAUNCH, "stream synchronize: %s", hipGetErrorString(e));
  for (int i = 0; i < h->prof_n; ++i) {
    e = hipEventElapsedTime(&ms_host[i], h->prof_ev[2 * i], h->prof_ev[2 * i + 1]);
    if (e != hipSuccess) return set_err(h, IM_ERR_LAUNCH, "hipEventElapsedTime: %s", hipGetErrorString(e));
  }
  *n_records = h->prof_n;
  release_profile(h);
  return IM_OK;
}

const char* im_last_error(const im_handle* h) { return h ? h->err : g_static_err; }

int32_t im_set_max_live(im_handle* h, int32_t max_live) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(max_live >= 1 && max_live <= h->cfg.capacity, "max_live must be in 1..capacity");
  h->max_live = max_live;
  return IM_OK;
}

int32_t im_query_status(im_handle* h, int32_t* status_host, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(status_host, "status_host is NULL");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(status_host, status_ptr(h), sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return set_err(h, IM_ERR_LAUNCH, "status copy: %s", hipGetErrorString(e));
  k_fill_i32<<<1, 64, 0, s>>>(status_ptr(h), 1, 0);
  rc = launch_check(h, "status clear");
  if (rc) return rc;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return set_err(h, IM_ERR_LAUNCH, "stream synchronize: %s", hipGetErrorString(e));
  return IM_OK;
}

int32_t im_append_kv(im_handle* h, const im_state* st, const void* k_new, const void* v_new,
                     const int32_t* pos_new, int32_t n_new, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(pos_new && ((k_new && v_new) || (!k_new && !v_new)), "pos_new is NULL, or only one of k_new / v_new is");
  IM_REQUIRE(n_new >= 1 && n_new <= h->cfg.capacity, "n_new must be in 1..capacity");
  if (h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_append_kv: head_shared = 1 takes im_append_kv_hidden");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  const int units = c.batch * c.n_kv_heads;
  dim3 grid((n_new * 16 + 255) / 256, units);
  k_append_rows<<<grid, 256, 0, s>>>((bf16_t*)st->K, (bf16_t*)st->V, st->pos, st->len,
                                     (const bf16_t*)k_new, (const bf16_t*)v_new, pos_new, n_new,
                                     c.n_kv_heads, 1, c.capacity, n_new <= 16 ? status_ptr(h) : nullptr);
  if (n_new > 16) k_append_len<<<(units + 255) / 256, 256, 0, s>>>(st->len, units, n_new, c.capacity, status_ptr(h));
  return launch_check(h, "im_append_kv");
}

int32_t im_append_kv_hidden(im_handle* h, const im_params* p, const im_state* st, const void* k_new,
                            const void* v_new, const void* x_new, const int32_t* pos_new,
                            int32_t n_new, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(params_ok(p), "params has a NULL pointer");
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(x_new && pos_new && ((k_new && v_new) || (!k_new && !v_new)),
             "x_new / pos_new is NULL, or only one of k_new / v_new is");
  IM_REQUIRE(n_new >= 1 && n_new <= h->cfg.capacity, "n_new must be in 1..capacity");
  if (!h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_append_kv_hidden: head_shared = 0 takes im_append_kv");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  const int units = c.batch * c.n_kv_heads;
  dim3 grid((n_new * 16 + 255) / 256, units);
  k_append_rows<<<grid, 256, 0, s>>>((bf16_t*)st->K, (bf16_t*)st->V, st->pos, st->len,
                                     (const bf16_t*)k_new, (const bf16_t*)v_new, pos_new, n_new,
                                     c.n_kv_heads, c.n_kv_heads, c.capacity, nullptr);
  double* xk = (double*)(h->ws + h->off_xk);
  const int M = c.batch * n_new;
  if (M <= 32)
    k_gemv_nt_f64<<<IM_DI_SHARED / 2, 256, 0, s>>>((const bf16_t*)x_new, (const bf16_t*)p->Uk, xk, M, IM_DI_SHARED,
                                                   c.gate_in_dim);
  else
    gemm_nt(s, (const bf16_t*)x_new, (const bf16_t*)p->Uk, xk, M, IM_DI_SHARED, c.gate_in_dim);
  k_store_hidden_keys<<<dim3((n_new + 15) / 16, c.batch), 256, 0, s>>>(
      xk, (bf16_t*)st->Kidx, st->len, st->n_projected, (const bf16_t*)p->norm_k_w, n_new, c.capacity, c.rms_eps);
  k_append_len<<<(c.batch + 255) / 256, 256, 0, s>>>(st->len, c.batch, n_new, c.capacity, status_ptr(h));
  return launch_check(h, "im_append_kv_hidden");
}

int32_t im_index_score(im_handle* h, const im_params* p, const im_state* st, const void* q_new,
                       const void* x_gate, const int32_t* q_pos, int32_t n_q, float* scores_out,
                       void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(params_ok(p), "params has a NULL pointer");
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(q_new && x_gate && q_pos && scores_out, "q_new / x_gate / q_pos / scores_out is NULL");
  IM_REQUIRE(n_q >= 1 && n_q <= h->cfg.max_queries, "n_q must be in 1..max_queries");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  const int units = n_sets(c), di = c.idx_dim;
  double* qy = (double*)(h->ws + h->off_qy);
  double* al = (double*)(h->ws + h->off_alpha);

  const int M = c.batch * n_q, Nq = c.n_idx_heads * di, Kq = c.n_q_heads * IM_D;
  const double alpha_denom = sqrt((double)(c.n_idx_heads * di));
  if (M <= 32) {
    // a decode-size call: the key projection of the new rows and both query-side products in one launch
    const int n_proj = c.head_shared ? 0 : units;
    k_query_side_few<<<n_proj * IM_PROJ_WGS + (Nq + 1) / 2 + (c.n_idx_heads + 1) / 2, 256, 0, s>>>(
        (const bf16_t*)q_new, (const bf16_t*)p->Uq, qy, Nq, Kq, (const bf16_t*)x_gate, (const bf16_t*)p->G, al,
        c.n_idx_heads, c.gate_in_dim, M, n_proj, (const bf16_t*)st->K, (bf16_t*)st->Kidx, st->len, st->n_projected,
        (const bf16_t*)p->Uk, (const bf16_t*)p->norm_k_w, c.capacity, h->max_live, c.rms_eps, status_ptr(h));
  } else {
    if (!c.head_shared)
      k_project_keys<<<dim3((h->max_live + 63) / 64, units), 256, 0, s>>>(
          (const bf16_t*)st->K, (bf16_t*)st->Kidx, st->len, st->n_projected, (const bf16_t*)p->Uk,
          (const bf16_t*)p->norm_k_w, c.capacity, h->max_live, c.rms_eps, status_ptr(h));
    if (c.gate_in_dim % 128 == 0 && gemm_tiles(M, Nq) <= 2048) {
      k_query_side<<<(M + 15) / 16 + gemm_tiles(M, Nq), 256, 0, s>>>(
          (const bf16_t*)q_new, (const bf16_t*)p->Uq, qy, M, Nq, Kq, (const bf16_t*)x_gate, (const bf16_t*)p->G, al,
          c.n_idx_heads, c.gate_in_dim);
    } else {
      if (n_q >= c.n_idx_heads && exact_fits(&c, M)) exact_project(h, s, (const bf16_t*)q_new, (const bf16_t*)p->Uq, qy, M);
      else gemm_nt(s, (const bf16_t*)q_new, (const bf16_t*)p->Uq, qy, M, Nq, Kq);
      gemm_nt(s, (const bf16_t*)x_gate, (const bf16_t*)p->G, al, M, c.n_idx_heads, c.gate_in_dim);
    }
  }
  // fewer queries than indexer heads (a decode step): the heads of a query are the scoring product's columns
  if (n_q < c.n_idx_heads) {
    // every wave normalises for itself (0.7 us a query) where few share a SIMD: 1176 waves 4.7 -> 6.9 us and a launch of 3.7
    // less, 4224 waves 8.5 -> 14.1; more queries or keys take k_qnorm_alpha
    const bool raw = n_q <= 4 && (long long)((h->max_live + 15) / 16) * units <= 2048;
    const int rows = M * c.n_idx_heads;
    if (!raw)
      k_qnorm_alpha<<<(rows + 3) / 4 + (rows + 255) / 256, 256, 0, s>>>(qy, rows, di, (const bf16_t*)p->norm_q_w,
                                                                       c.rms_eps, al, rows, alpha_denom);
    const dim3 grid((h->max_live + 63) / 64, units);
#define IM_SCORE_FEW(DI, RAW)                                                                                       \
  k_score_few<DI, RAW><<<grid, 256, 0, s>>>((const bf16_t*)st->Kidx, st->pos, st->len, st->n_projected, qy, al, q_pos, \
                                            n_q, c.n_kv_heads / heads_per_set(c), c.capacity, c.n_idx_heads,        \
                                            h->max_live, (const bf16_t*)p->norm_q_w, c.rms_eps, alpha_denom, scores_out)
    if (c.head_shared) { if (raw) IM_SCORE_FEW(IM_DI_SHARED, true); else IM_SCORE_FEW(IM_DI_SHARED, false); }
    else { if (raw) IM_SCORE_FEW(IM_DI, true); else IM_SCORE_FEW(IM_DI, false); }
#undef IM_SCORE_FEW
    return launch_check(h, "im_index_score");
  }
  const bf16_t* nqw = (const bf16_t*)p->norm_q_w;
  if (score_short(h, n_q)) {
    const int rows = M * c.n_idx_heads;
    k_qnorm_alpha<<<(rows + 3) / 4 + (rows + 255) / 256, 256, 0, s>>>(qy, rows, di, nqw, c.rms_eps, al, rows, alpha_denom);
    // few (256-key tile, unit) workgroups: a group of queries per workgroup; very few: 16 keys per wave instead of 64, too
    const bool small = score_tiles(h) < 128;
    const int nblk = (n_q + 15) / 16, per_group = score_tiles(h) < IM_SCORE_GROUP_TILES ? (nblk + IM_SCORE_GROUPS - 1) / IM_SCORE_GROUPS * 16 : n_q;
    const int groups = (n_q + per_group - 1) / per_group, live = h->max_live;
    float* out = groups > 1 ? (float*)(h->ws + h->off_spart) : scores_out;
#define IM_SCORE(TPW, DI)                                                                                          \
  k_score<TPW, DI><<<dim3((live + 64 * TPW - 1) / (64 * TPW), units, groups), 256, 0, s>>>(                        \
      (const bf16_t*)st->Kidx, st->pos, st->len, st->n_projected, qy, al, q_pos, n_q, c.n_kv_heads / heads_per_set(c), \
      c.capacity, c.n_idx_heads, live, out, groups > 1 ? live : c.capacity, per_group)
    if (c.head_shared) { if (small) IM_SCORE(1, IM_DI_SHARED); else IM_SCORE(4, IM_DI_SHARED); }
    else { if (small) IM_SCORE(1, IM_DI); else IM_SCORE(4, IM_DI); }
#undef IM_SCORE
    if (groups > 1)
      k_score_max<<<dim3((live + 255) / 256, units), 256, 0, s>>>(out, groups, st->len, c.capacity, live, scores_out);
    return launch_check(h, "im_index_score");
  }
  if (c.head_shared) {
    if (c.n_idx_heads <= 8) score_many<IM_DI_SHARED, 8>(h, st, nqw, q_pos, n_q, alpha_denom, scores_out, s);
    else score_many<IM_DI_SHARED, 16>(h, st, nqw, q_pos, n_q, alpha_denom, scores_out, s);
  } else {
    if (c.n_idx_heads <= 8) score_many<IM_DI, 8>(h, st, nqw, q_pos, n_q, alpha_denom, scores_out, s);
    else score_many<IM_DI, 16>(h, st, nqw, q_pos, n_q, alpha_denom, scores_out, s);
  }
  return launch_check(h, "im_index_score");
}

int32_t im_topb_select(im_handle* h, const float* scores, const im_state* st, int32_t budget,
                       int32_t* keep_idx, int32_t* evict_idx, int32_t* n_keep, int32_t* n_evict,
                       void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(scores && keep_idx && evict_idx && n_keep && n_evict, "an array pointer is NULL");
  IM_REQUIRE(budget >= h->cfg.n_sink + h->cfg.n_recent, "budget is below n_sink + n_recent");
  IM_REQUIRE(budget <= h->cfg.capacity, "budget exceeds capacity");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  const int live = h->max_live;
#define IM_SELECT(R)                                                                                               \
  k_select<R><<<n_sets(c), 1024, 0, s>>>(scores, st->pos, st->len, c.capacity, live, budget, c.n_sink, c.n_recent, \
                                         keep_idx, evict_idx, n_keep, n_evict, status_ptr(h))
  if (live <= 4 * 1024) IM_SELECT(4);
  else if (live <= 8 * 1024) IM_SELECT(8);
  else if (live <= 16 * 1024) IM_SELECT(16);
  else IM_SELECT(0);
#undef IM_SELECT
  return launch_check(h, "im_topb_select");
}

int32_t im_memory_update(im_handle* h, const im_params* p, const im_state* st,
                         const int32_t* evict_idx, const int32_t* n_evict, float lambda, float eta,
                         void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(params_ok(p), "params has a NULL pointer");
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(evict_idx && n_evict, "evict_idx / n_evict is NULL");
  IM_REQUIRE(lambda > 0.f && lambda <= 1.f, "lambda must be in (0, 1]");
  IM_REQUIRE(eta > 0.f, "eta must be > 0");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  const int units = n_sets(c);
  float* part = (float*)(h->ws + h->off_mem);
  // (a tile of a set holds the rows of all its heads: its splits may be shorter than a fold block)
  const int n_split = mem_splits(&c, h->max_live), fold = c.head_shared ? IM_MEM_TOK : c.fold_block;
  if (c.head_shared)
    k_mem_partial_sets<<<dim3(units, n_split), 256, 0, s>>>(
        (const bf16_t*)st->K, (const bf16_t*)st->V, evict_idx, n_evict, (const bf16_t*)p->Wtheta,
        c.capacity, c.n_kv_heads, fold, n_split, part);
  else
    k_mem_partial<<<dim3(units, n_split), 256, 0, s>>>(
        (const bf16_t*)st->K, (const bf16_t*)st->V, evict_idx, n_evict, (const bf16_t*)p->Wtheta,
        c.capacity, fold, n_split, part);
  k_mem_finalize<<<dim3((IM_DM * IM_D + IM_DM + 255) / 256, units), 256, 0, s>>>(
      st->M, st->b, n_evict, part, fold, n_split, lambda, eta, (const bf16_t*)st->K,
      (const bf16_t*)st->V, evict_idx, (const bf16_t*)p->Wtheta, c.capacity, heads_per_set(c));
  return launch_check(h, "im_memory_update");
}

int32_t im_compact_kv(im_handle* h, const im_state* st, const int32_t* keep_idx, const int32_t* n_keep,
                      const int32_t* evict_idx, const int32_t* n_evict, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(keep_idx && n_keep && evict_idx && n_evict, "a list pointer is NULL");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  int gx = (h->max_live + 3) / 4;
  if (gx > 64) gx = 64;
  k_compact<<<dim3(gx, c.batch * c.n_kv_heads), 256, 0, s>>>(
      (bf16_t*)st->K, (bf16_t*)st->V, (bf16_t*)st->Kidx, st->pos, st->len, st->n_projected, keep_idx,
      n_keep, evict_idx, n_evict, c.capacity, heads_per_set(c), c.idx_dim, h->max_live, status_ptr(h));
  return launch_check(h, "im_compact_kv");
}

int32_t im_gather_kept(im_handle* h, const im_state* src, const im_state* dst, int32_t dst_capacity,
                       const int32_t* keep_idx, const int32_t* n_keep, const int32_t* evict_idx,
                       const int32_t* n_evict, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(state_ok(src) && state_ok(dst), "a state has a NULL pointer");
  IM_REQUIRE(keep_idx && n_keep && evict_idx && n_evict, "a list pointer is NULL");
  IM_REQUIRE(dst_capacity >= 1, "dst_capacity must be >= 1");
  IM_REQUIRE(src->K != dst->K && src->V != dst->V && src->Kidx != dst->Kidx && src->pos != dst->pos &&
                 src->M != dst->M && src->b != dst->b,
             "source and destination must be different buffers (im_compact_kv works in place)");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  const im_config& c = h->cfg;
  int gx = (h->max_live + 3) / 4;
  if (gx > 64) gx = 64;
  k_gather_kept<<<dim3(gx, c.batch * c.n_kv_heads), 256, 0, s>>>(
      (const bf16_t*)src->K, (const bf16_t*)src->V, (const bf16_t*)src->Kidx, src->pos, src->len, src->M, src->b,
      (bf16_t*)dst->K, (bf16_t*)dst->V, (bf16_t*)dst->Kidx, dst->pos, dst->len, dst->n_projected, dst->M, dst->b,
      keep_idx, n_keep, evict_idx, c.capacity, dst_capacity, heads_per_set(c), c.idx_dim, h->max_live, status_ptr(h));
  return launch_check(h, "im_gather_kept");
}

// the two launches of step a5 over `part` (attention partials, attn_chunks records per query head)
static int launch_attn(const im_config& c, int max_live, const im_params* p, const im_state* st, const void* q,
                       void* out, float* readout_dbg, float* part, int attn_chunks, int32_t* status,
                       hipStream_t s) {
  const int units = c.batch * c.n_kv_heads, G = c.n_q_heads / c.n_kv_heads;
  const int H_set = c.head_shared ? c.n_kv_heads : 1;
  const int chunks = (max_live + IM_ATT_CHUNK - 1) / IM_ATT_CHUNK;
  dim3 grid(chunks, units);
#define IM_ATT_CASE(g)                                                                          \
  case g:                                                                                       \
    k_attn_partial<g><<<grid, 256, 0, s>>>((const bf16_t*)st->K, (const bf16_t*)st->V, st->len,   \
                                           (const bf16_t*)q, c.n_q_heads, c.n_kv_heads, H_set,   \
                                           c.capacity, max_live, c.softmax_scale, part,         \
                                           attn_chunks, status);                                \
    break;
  switch (G) {
    IM_ATT_CASE(1) IM_ATT_CASE(2) IM_ATT_CASE(3) IM_ATT_CASE(4)
    IM_ATT_CASE(5) IM_ATT_CASE(6) IM_ATT_CASE(7) IM_ATT_CASE(8)
    default: return IM_ERR_UNSUPPORTED;
  }
#undef IM_ATT_CASE
  k_attn_combine<<<c.batch * c.n_q_heads, 128, 0, s>>>(
      part, attn_chunks, st->len, (const bf16_t*)q, (const bf16_t*)p->Wtheta, (const bf16_t*)p->wg,
      p->cg, st->M, st->b, c.n_q_heads, c.n_kv_heads, H_set, max_live, c.mem_eps, (bf16_t*)out,
      readout_dbg);
  return IM_OK;
}

int32_t im_decode_attn_with_readout(im_handle* h, const im_params* p, const im_state* st,
                                    const void* q, void* out, float* readout_dbg, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(params_ok(p), "params has a NULL pointer");
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(q && out, "q / out is NULL");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  rc = launch_attn(h->cfg, h->max_live, p, st, q, out, readout_dbg, (float*)(h->ws + h->off_attn),
                   h->attn_chunks, status_ptr(h), s);
  if (rc) return set_err(h, rc, "group size %d", h->cfg.n_q_heads / h->cfg.n_kv_heads);
  return launch_check(h, "im_decode_attn_with_readout");
}

static size_t static_scratch_bytes(const im_config* cfg, int32_t max_live) {
  int code;
  if (config_problem(cfg, &code) || max_live < 1 || max_live > cfg->capacity) return 0;
  const size_t chunks = ((size_t)max_live + IM_ATT_CHUNK - 1) / IM_ATT_CHUNK;
  return 256 + (size_t)cfg->batch * cfg->n_q_heads * chunks * IM_ATT_REC * sizeof(float);
}

int32_t im_decode_attn_with_readout_static(const im_config* cfg, int32_t max_live, const im_params* p,
                                           const im_state* st, const void* q, void* out,
                                           float* readout_dbg, int32_t* status_dev, void* stream) {
  // host-only validation first: an invalid call touches no GPU
  int code;
  if (const char* why = config_problem(cfg, &code)) return static_err(code, "im_decode_attn_with_readout_static: %s", why);
  if (!params_ok(p) || !state_ok(st) || !q || !out)
    return static_err(IM_ERR_INVALID_ARG, "im_decode_attn_with_readout_static: a params / state / q / out pointer is NULL");
  if (max_live < 1 || max_live > cfg->capacity)
    return static_err(IM_ERR_INVALID_ARG, "im_decode_attn_with_readout_static: max_live must be in 1..capacity");
  const size_t need = static_scratch_bytes(cfg, max_live);
  if (need > (size_t)IM_STATIC_SCRATCH_BYTES)
    return static_err(IM_ERR_INVALID_ARG,
                      "im_decode_attn_with_readout_static: batch %d x %d query heads x %d live entries need %zu bytes of "
                      "scratch, the built-in buffer holds %zu (IM_STATIC_SCRATCH_BYTES); use im_decode_attn_with_readout "
                      "with a workspace",
                      cfg->batch, cfg->n_q_heads, max_live, need, (size_t)IM_STATIC_SCRATCH_BYTES);
  // this device's copy of the scratch array: looked up once per device, with that device current
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= IM_STATIC_MAX_DEVICES)
    return static_err(IM_ERR_LAUNCH, "im_decode_attn_with_readout_static: hipGetDevice: %s (device %d)",
                      hipGetErrorString(e), dev);
  char* scratch = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
      void* sym = nullptr;
      e = hipGetSymbolAddress(&sym, HIP_SYMBOL(im_static_scratch));
      if (e != hipSuccess || !sym)
        return static_err(IM_ERR_LAUNCH, "im_decode_attn_with_readout_static: hipGetSymbolAddress: %s",
                          hipGetErrorString(e));
      g_static_ptr[dev] = sym;
    }
    scratch = (char*)g_static_ptr[dev];
  }
  hipStream_t s = (hipStream_t)stream;
  // the buffer keeps the last call's contents.  The partial records need no clearing (every record the
  // combine reads is written by this call's first launch); the status word does when it is the sink.
  int32_t* status = status_dev ? status_dev : (int32_t*)scratch;
  if (!status_dev) k_fill_i32<<<1, 64, 0, s>>>((int32_t*)scratch, 1, 0);
  const int chunks = (max_live + IM_ATT_CHUNK - 1) / IM_ATT_CHUNK;
  const int rc = launch_attn(*cfg, max_live, p, st, q, out, readout_dbg, (float*)(scratch + 256), chunks, status, s);
  if (rc) return static_err(rc, "im_decode_attn_with_readout_static: group size %d", cfg->n_q_heads / cfg->n_kv_heads);
  e = hipGetLastError();
  if (e != hipSuccess) return static_err(IM_ERR_LAUNCH, "im_decode_attn_with_readout_static: %s", hipGetErrorString(e));
  return IM_OK;
}

static int32_t decode_launch(im_handle* h, const im_params* p, const im_state* st, const void* q,
                             const void* x_gate, const int32_t* q_pos, const void* k_new, const void* v_new,
                             const int32_t* pos_new, int32_t budget, float lambda, float eta, void* out,
                             float* readout_dbg, int32_t* evicted_slot, float* scores_dbg, void* stream,
                             const bool no_score, const int32_t* ext_evict, const char* what) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(params_ok(p), "params has a NULL pointer");
  IM_REQUIRE(state_ok(st), "state has a NULL pointer");
  IM_REQUIRE(q && k_new && v_new && pos_new && out, "an input / output pointer is NULL");
  IM_REQUIRE(no_score || (x_gate && q_pos), "x_gate / q_pos is NULL");
  IM_REQUIRE(!h->cfg.head_shared || x_gate, "the new token's hidden state is NULL");
  IM_REQUIRE(budget >= h->cfg.n_sink + h->cfg.n_recent, "budget is below n_sink + n_recent");
  IM_REQUIRE(budget <= h->cfg.capacity, "budget exceeds capacity");
  IM_REQUIRE(lambda > 0.f && lambda <= 1.f, "lambda must be in (0, 1]");
  IM_REQUIRE(eta > 0.f, "eta must be > 0");
  const im_config& c = h->cfg;
  if (c.batch > 64) return set_err(h, IM_ERR_UNSUPPORTED, "%s: batch above 64", what);
  if (c.head_shared && h->max_live > 64 * DEC_KEYS + 1)
    return set_err(h, IM_ERR_UNSUPPORTED, "%s: head_shared = 1 needs max_live <= %d", what, 64 * DEC_KEYS + 1);
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_ws(h, s);
  if (rc) return rc;
  if (c.head_shared && c.n_kv_heads > 16)
    return set_err(h, IM_ERR_UNSUPPORTED, "%s: head_shared = 1 with more than 16 KV heads", what);
  const int units = c.batch * c.n_kv_heads, G = c.n_q_heads / c.n_kv_heads;
  int32_t* words = (int32_t*)(h->ws + h->off_status);
  DecArgs a = {};
  a.K = (bf16_t*)st->K; a.V = (bf16_t*)st->V; a.Kidx = (bf16_t*)st->Kidx;
  a.pos = st->pos; a.len = st->len; a.nproj = st->n_projected; a.M = st->M; a.bvec = st->b;
  a.Uq = (const bf16_t*)p->Uq; a.Gw = (const bf16_t*)p->G; a.Uk = (const bf16_t*)p->Uk;
  a.nqw = (const bf16_t*)p->norm_q_w; a.nkw = (const bf16_t*)p->norm_k_w;
  a.Wt = (const bf16_t*)p->Wtheta; a.wg = (const bf16_t*)p->wg; a.cg = p->cg;
  a.q = (const bf16_t*)q; a.xg = (const bf16_t*)x_gate; a.k_new = (const bf16_t*)k_new;
  a.v_new = (const bf16_t*)v_new; a.pos_new = pos_new; a.q_pos = q_pos; a.named = ext_evict;
  a.out = (bf16_t*)out; a.readout = readout_dbg; a.scores = scores_dbg; a.evicted = evicted_slot;
  a.qy = (double*)(h->ws + h->off_qy); a.alpha = (double*)(h->ws + h->off_alpha);
  a.status = words; a.maxpos = words + 32; a.arrived = (int32_t*)(h->ws + h->off_darrived);
  a.part = (float*)(h->ws + h->off_dpart); a.part_ml = (float2*)(h->ws + h->off_dml);
  a.qm = (float*)(h->ws + h->off_dqm); a.pick = (uint4*)(h->ws + h->off_dpick);
  a.xk = (double*)(h->ws + h->off_xk);
  a.B = c.batch; a.H = c.n_q_heads; a.H_kv = c.n_kv_heads; a.C = c.capacity; a.H_idx = c.n_idx_heads;
  a.gate_in = c.gate_in_dim; a.n_sink = c.n_sink; a.n_recent = c.n_recent; a.budget = budget;
  // 128-key splits over all live entries but the last, which the second launch takes
  a.S = h->max_live > 1 ? (h->max_live - 1 + DEC_KEYS - 1) / DEC_KEYS : 1;
  a.max_live = h->max_live;
  a.rms_eps = c.rms_eps; a.mem_eps = c.mem_eps; a.scale = c.softmax_scale; a.lambda = lambda; a.eta = eta;
  a.G = G; a.kv_magic = (uint32_t)((1ull << 32) / (unsigned)c.n_kv_heads) + 1u;
  a.alpha_denom = sqrt((double)(c.n_idx_heads * c.idx_dim));
  a.hs = c.head_shared; a.H_set = heads_per_set(c); a.di = c.idx_dim; a.score = no_score ? 0 : 1;
  // projection blocks take two weight rows (U_q and G where the step scores, U_k in the head-shared layout) and 4 batch rows each (a
  // shorter chain per block) while the roles then still are one generation of workgroups (4 per CU), else 8: 16 sequences x 4 heads,
  // 32 layer-steps 845 us with 4, 802 with 8
  const int row_pairs = (a.score ? c.n_idx_heads * c.idx_dim / 2 + (c.n_idx_heads + 1) / 2 : 0) + (a.hs ? IM_DI_SHARED / 2 : 0);
  const int prep_rows = a.score && row_pairs * ((c.batch + 3) / 4) + (1 + DEC_MP) * units > 4 * 256 ? 8 : 4;
  a.n_proj = row_pairs * ((c.batch + prep_rows - 1) / prep_rows);
  const int n_roles = ((1 + DEC_MP) * units + a.n_proj + 7) / 8 * 8;
  // 16-key tiles per wave of the scoring launch: a wave's fixed chain is paid once for its tiles, and few waves leave SIMDs without one.
  // Passes over 32 layer-steps with 1, 2, 4 tiles, us: 1312 tiles in all 550, 560, 555; 1824: 602, 588, 617; 2080: 603, 597, 610; 2056
  // (8 sets): 640, 592, 598; 2112 (64 sets) 786, 783, 801; 4128: 830, 748, 725.  With more than 8 indexer heads a tile is twice the work, and
  // there are 1 or 2; us per layer-step with 1, 2 (64 query heads): 520 tiles in all 19.4, 20.0; 1032: 21.8, 21.6; 1056: 21.5, 22.1; 1704: 23.9,
  // 21.9; 2056: 25.2, 23.9; 4128: 31.4, 28.4; 8704: 112.8, 110.0.  Head-shared, where a tile is a quarter of the work, 2 or 4; us per layer-step
  // with 1, 2, 4: 129 tiles in all 15.4, 15.0, 15.0; 516: 20.3, 20.2, 20.4; 903: 27.5, 25.5, 25.6; 1040: 32.0, 30.6, 30.7; 1560: 39.7, 40.1, 40.3; 2080: 48.6,
  // 48.1, 48.2; 4160: 86.5, 85.1, 84.5; 64 query heads, 1040: 39.2, 37.9, 37.8
  const long long key_tiles = (long long)n_sets(c) * ((h->max_live + 15) / 16);
  int tiles = key_tiles > 3072 ? 4 : key_tiles > 1536 ? 2 : 1;
  if (c.head_shared) tiles = max(tiles, 2);
  else if (c.n_idx_heads > 8) tiles = min(tiles, 2);
  a.n_pick = a.score ? (a.max_live + 16 * tiles - 1) / (16 * tiles) : 0;
  const bool prof = h->prof_ev && h->prof_n < h->prof_max;
  hipEvent_t ev0 = prof ? h->prof_ev[2 * h->prof_n] : nullptr, ev1 = prof ? h->prof_ev[2 * h->prof_n + 1] : nullptr;
  // what a step of three launches brackets: the first, the second, or both; of two launches the first
  hipEvent_t mid = nullptr, end = nullptr;
  if (prof) {
    const bool three = a.score != 0;
    if (!three || h->prof_span != IM_PROFILE_MAIN) (void)hipEventRecord(ev0, s);
    if (three && h->prof_span == IM_PROFILE_MAIN) mid = ev0;
    if (three && h->prof_span == IM_PROFILE_PREP) mid = ev1; else end = ev1;
  }
  launch_step(a, n_roles, prep_rows, tiles, mid, end, s);
  if (prof) h->prof_n++;
  return launch_check(h, what);
}

int32_t im_decode_step(im_handle* h, const im_params* p, const im_state* st, const void* q,
                       const void* x_gate, const int32_t* q_pos, const void* k_new, const void* v_new,
                       const int32_t* pos_new, int32_t budget, float lambda, float eta, void* out,
                       float* readout_dbg, int32_t* evicted_slot, float* scores_dbg, void* stream) {
  return decode_launch(h, p, st, q, x_gate, q_pos, k_new, v_new, pos_new, budget, lambda, eta, out,
                       readout_dbg, evicted_slot, scores_dbg, stream, false, nullptr, "im_decode_step");
}

int32_t im_attend_step(im_handle* h, const im_params* p, const im_state* st, const void* q,
                       const void* k_new, const void* v_new, const int32_t* pos_new, void* out,
                       float* readout_dbg, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  // budget = capacity: no unit can be above it, so nothing is evicted; lambda, eta are unused
  if (h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_attend_step: head_shared = 1 takes im_attend_step_hidden");
  return decode_launch(h, p, st, q, nullptr, nullptr, k_new, v_new, pos_new, h->cfg.capacity, 1.f, 1.f, out,
                       readout_dbg, nullptr, nullptr, stream, true, nullptr, "im_attend_step");
}

int32_t im_attend_step_hidden(im_handle* h, const im_params* p, const im_state* st, const void* q,
                              const void* x_new, const void* k_new, const void* v_new,
                              const int32_t* pos_new, void* out, float* readout_dbg, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  if (!h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_attend_step_hidden: head_shared = 0 takes im_attend_step");
  return decode_launch(h, p, st, q, x_new, nullptr, k_new, v_new, pos_new, h->cfg.capacity, 1.f, 1.f, out,
                       readout_dbg, nullptr, nullptr, stream, true, nullptr, "im_attend_step_hidden");
}

int32_t im_decode_step_shared(im_handle* h, const im_params* p, const im_state* st, const void* q,
                              const void* k_new, const void* v_new, const int32_t* pos_new,
                              const int32_t* evict_slot, float lambda, float eta, void* out,
                              float* readout_dbg, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(evict_slot, "evict_slot is NULL");
  if (h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_decode_step_shared: head_shared = 1 takes im_decode_step_shared_hidden");
  return decode_launch(h, p, st, q, nullptr, nullptr, k_new, v_new, pos_new, h->cfg.capacity, lambda, eta, out,
                       readout_dbg, nullptr, nullptr, stream, true, evict_slot, "im_decode_step_shared");
}

int32_t im_decode_step_shared_hidden(im_handle* h, const im_params* p, const im_state* st, const void* q,
                                     const void* x_new, const void* k_new, const void* v_new,
                                     const int32_t* pos_new, const int32_t* evict_slot, float lambda,
                                     float eta, void* out, float* readout_dbg, void* stream) {
  if (!h) return IM_ERR_INVALID_ARG;
  IM_REQUIRE(evict_slot, "evict_slot is NULL");
  if (!h->cfg.head_shared) return set_err(h, IM_ERR_UNSUPPORTED, "im_decode_step_shared_hidden: head_shared = 0 takes im_decode_step_shared");
  return decode_launch(h, p, st, q, x_new, nullptr, k_new, v_new, pos_new, h->cfg.capacity, lambda, eta, out,
                       readout_dbg, nullptr, nullptr, stream, true, evict_slot, "im_decode_step_shared_hidden");
}

}  // extern "C"
