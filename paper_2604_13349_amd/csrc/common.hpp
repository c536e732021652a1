// Internal declarations shared by the translation units of libobf_relay.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <mutex>
#include "obf_relay.h"

namespace obf {

constexpr int kMaxTokens = 32768;
constexpr int kNumCU = 256;             // compute units of the target (MI355X)
constexpr int kStatChunk = 1024;        // tokens per deleted-value statistics workgroup
constexpr int kGatherRows = 64;         // rows per gather workgroup when a row is 256 bytes (bf16, head_dim 128)
constexpr int kBandCap = 256;           // most boundary candidates re-scored per head
constexpr double kEps = 1e-12;          // epsilon of Eq. 4 / Eq. 6
constexpr float kBandRel = 1.0e-4f;     // relative half-width of the refinement band

struct Dims {
  int heads;      // n_layers * n_kv_heads
  int L, H, g, d, N, W;
  int kvs;        // tokens between consecutive heads of K and V (>= N; N for a dense cache)
  int scs;        // floats between consecutive heads of the score array handed to selection and back-fill (>= N)
  int R;          // query rows per KV head = g * W
  int dtype;
  int esize;      // bytes per element of K/V/Q
};

inline Dims make_dims(const obf_shape_t* s) {
  Dims m;
  m.L = s->n_layers; m.H = s->n_kv_heads; m.g = s->group; m.d = s->head_dim; m.N = s->n_tokens; m.W = s->window;
  m.kvs = m.N; m.scs = m.N;
  m.heads = m.L * m.H; m.R = m.g * m.W; m.dtype = s->dtype; m.esize = (s->dtype == OBF_BF16) ? 2 : 4;
  return m;
}

// Heads with many retained rows that the full-rank certificate does not settle (rare): the double-precision Gram
// matrix of their rows is summed from kKeepGramChunks partial matrices computed by as many workgroups, for at most
// kKeepGramSlots such heads per call (further ones compute it in their own workgroup); used from kKeepGramMinBudget rows.
constexpr int kJacobiSweeps = 12;       // cap of the cyclic Jacobi iteration of the finalisation
constexpr int kKeepGramChunks = 16;
constexpr int kKeepGramSlots = 8;
constexpr int kKeepGramMinBudget = 2048;

// Query rows per workgroup of the matrix-core score kernels: 128 (four 32-row blocks) or 160 (five), whichever pads the
// g * W rows of a KV head less; ties go to 128, which has one more K buffer in flight.
inline int score_rows_per_group(int R) {
  const int g4 = (R + 127) / 128, g5 = (R + 159) / 160;
  return (g5 * 160 - R < g4 * 128 - R) ? 160 : 128;
}

// 32-token tiles per persistent workgroup of those kernels, TT in all: as many ranges as make a multiple of 8 (one share per XCD) such that an
// XCD's ranges x row groups fit its 32 compute units.
inline int score_tiles_per_range(long TT, int rgroups) {
  const int per_xcd = (kNumCU / 8) / rgroups > 0 ? (kNumCU / 8) / rgroups : 1;
  const int G = 8 * per_xcd;
  long T = (TT + G - 1) / G;
  T = ((T + 3) / 4) * 4;
  return (int)(T < 4 ? 4 : T);
}

// Rows per group of the score kernels that carry 192 or 256 rows (score_tall.hip), 0 where those of 128 or 160 pad less (257 to 320 rows: two groups
// of 160) or one such group holds all rows.
inline int score_tall_rows(int R) {
  if (R <= 160) return 0;
  const int g = score_rows_per_group(R), narrow = (R + g - 1) / g * g;
  const int p192 = (R + 191) / 192 * 192, p256 = (R + 255) / 256 * 256;
  const int wide = p192 < p256 ? p192 : p256;
  return wide > narrow ? 0 : p192 < p256 ? 192 : 256;
}
constexpr int kScoreTallStep = 64;       // tokens per step of them

// Workspace carving.  Every region is 256-byte aligned; offsets are from the workspace base.
struct Workspace {
  size_t stats_part;   // double2 [heads][nchunk][R]      partial (max, sum-exp) per score chunk
  size_t row_lse;      // double  [heads][R]
  size_t scores;       // float   [heads][N]              (fused call without scores_out)
  size_t score_part;   // float   [rgroups - 1][heads][N] column sums of all row groups but the last, whose lie where the scores will
  size_t head_state;   // HeadState [heads]
  size_t decided;      // int32   [heads]                 1: the fast full-rank test settled the head
  size_t basis;        // float   [heads][d][d]           orthonormal basis of the retained span (columns)
  size_t gram_part;    // float   [heads][nstat][gram_stride(d)] partial Gram / weighted sum / plain sum / norm of V_del
  size_t mats;         // float   [heads][3][d*d]         scratch matrices of the per-head finalisation
  size_t delta;        // float   [heads][d]
  size_t sel_flags;    // int32   [heads]: OBF_SELECT_* bits of the fused selection (read into obf_diag_t when diagnostics are asked for)
  size_t band;         // 16 bytes [heads][kBandCap]: scratch of the threshold re-decision (layerwise: exact per-head masses of the band)
  size_t layer_scores; // float   [L][N]        attention mass summed over the heads of a layer (layerwise selector)
  size_t layer_idx;    // int32   [L][max_budget], then int32 [L]: the shared index lists and their lengths
  size_t fro_part;     // double  [heads][ceil(max_budget/16)]   per-gather-block sums of squares of the retained V rows
  size_t keep_gram;    // double  [kKeepGramSlots][kKeepGramChunks][d*d]  partial Gram matrices (max_budget >= kKeepGramMinBudget)
  size_t rot;          // float   [heads][kJacobiSweeps][d-1][d/2]  rotation tangents of the Jacobi iteration (max_budget < d only)
  size_t inv_norm;     // float   [heads][max_budget]     reciprocal norms of the retained keys (cache merging)
  size_t route;        // int32   [heads][N]              retained slot of every deleted token (cache merging, when not an output)
  size_t total;
  size_t lead_total;   // what a fused call needs whose back-fill takes at most kLeadMaxRank directions by the rank rule: all but the three regions before
  int nchunk;          // most chunks per head of the double-precision score path
  int tall_rows;       // 192 or 256: scores with row groups of that many; 0: others
  int rgroups, tiles_per_head, tiles_per_range, nranges;       // matrix-core score partition (tiles of 32 tokens, or steps of 64 with tall row groups)
  bool narrow_stats;   // tall row groups, but the first pass takes 128 rows at a time, on a partition of its own:
  int stats_rgroups, stats_tiles_per_head, stats_tiles_per_range, stats_nranges;
  int nslot;           // of the first pass: ranges that can meet in a head
  int nstat;           // statistics chunks per head
};

struct HeadState {
  double a_keep, a_del;
  int32_t n_keep, n_del;
  int32_t r_keep;       // dimension of the retained span, -1 = not computed
  int32_t active;       // 1: residual statistics and injection are needed
  int32_t k_used;
  int32_t pad;
  float rcr, ivn;
};

// One chunk's statistics of the deleted values: G [d][d] (tiles on and below the diagonal), u = sum_j A_j v_j [d],
// s = sum_j v_j [d], ||V_del||_F^2, padding.
__host__ __device__ inline size_t gram_stride(int d) { return (size_t)d * d + 2 * (size_t)d + 4; }

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline Workspace carve(const Dims& m, int max_budget, int rank) {
  Workspace w;
  // double-precision score path: at most one chunk per 512 tokens (or nslot below, whichever is more)
  w.nchunk = (m.N + 511) / 512;
  w.nstat = (m.N + kStatChunk - 1) / kStatChunk;
  // matrix-core score path: the flattened (head, 32-token tile) space is cut into one range per
  // persistent workgroup; a head is covered by at most nslot ranges
  int tall = m.dtype == OBF_BF16 && m.d == 128 ? score_tall_rows(m.R) : 0;
  // Two groups of 192 rows for three of 128 pad nothing less.  They are ahead by their shorter way from head to head; where a workgroup has
  // thousands of tokens of long heads, three are (both passes, 384 rows, us, three and two: 64 heads of 4096, 8192, 24000 tokens 81 - 72, 130 - 127,
  // 349 - 376; 288 of 2048, 4096, 8192, 20000 tokens 176 - 147, 302 - 284, 573 - 588, 1358 - 1440), and so nine for six (1152 rows: 64 heads of 2048 and
  // 96 of 32768 135 - 108, 2066 - 2167).
  bool sums_aside = false;                                      // the column sums lie in the bases, statistics and matrices, too
  if (tall == 192) {
    const int g = (m.R + 191) / 192, g128 = (m.R + 127) / 128;
    if (g128 * 128 <= g * 192 && m.N >= 8192 && (long)m.heads * m.N >= 4096L * 8 * (g < 64 ? 64 / g : 1)) {
      const bool more = g128 - 1 > g;                           // sets than six groups' were
      if (!more || (size_t)(g128 - 1) * m.N <= 4 * (size_t)m.d * m.d + w.nstat * gram_stride(m.d)) { tall = 0; sums_aside = more; }
    }
  }
  w.tall_rows = tall;
  const int group_rows = tall ? tall : score_rows_per_group(m.R);
  w.rgroups = (m.R + group_rows - 1) / group_rows;
  w.narrow_stats = false;
  auto slots = [](int per_head, int per_range) { return (per_head + per_range - 1) / per_range + 1; };
  int held = w.nchunk;                                          // slots that stats_part has room for
  if (tall) {                                                   // two workgroups per compute unit
    // Few heads are cut into more ranges than 128 rows at a time would be.  What their partials need beyond the room for those lies in the bases,
    // statistics and matrices of the back-fill, which are written after the scores; ranges grow where that is not enough either.
    const int tiles = (m.N + 31) / 32, per_old = score_tiles_per_range((long)m.heads * tiles, (m.R + score_rows_per_group(m.R) - 1) / score_rows_per_group(m.R));
    held = slots(tiles, per_old) > held ? slots(tiles, per_old) : held;
    const size_t spare = sizeof(float) * (4 * (size_t)m.d * m.d + w.nstat * gram_stride(m.d)) / (2 * sizeof(double) * (size_t)m.R);   // per head
    const int most = spare > (size_t)held ? (int)spare : held;
    w.tiles_per_head = (m.N + kScoreTallStep - 1) / kScoreTallStep;
    const long TT = (long)m.heads * w.tiles_per_head;
    const int per_xcd = (2 * kNumCU / 8) / w.rgroups > 0 ? (2 * kNumCU / 8) / w.rgroups : 1;
    w.tiles_per_range = (int)((TT + 8 * per_xcd - 1) / (8 * per_xcd));
    while (slots(w.tiles_per_head, w.tiles_per_range) > most) ++w.tiles_per_range;
    // Every workgroup of the second pass folds all partials of its head, 0.3 us each, and again where its range goes on into the next head; a step
    // costs both passes 3 us.  So few heads are cut into no more than 4 sqrt(steps) ranges each, and ranges end with their head (whose last one is the
    // shorter) where that makes them at most two steps longer, with one of them to a compute unit in place of two where that costs four more at
    // most.  Both passes, 192 rows (us), before, ranges of equal length that fill the card, and with this: 2 heads of 16384 and 32768 tokens 72, 73 - 27, 35;
    // 4 of 8192 44 - 23; 8 of 4096 and 16384 30, 39 - 19, 32; 24 of 4096 38 - 27; 96 of 1300 37 - 31; 160 of 2048 56 - 52; 288 of 256 31 - 26.
    const int SH = w.tiles_per_head, fit = 8 * per_xcd / m.heads;
    while (16L * w.tiles_per_range * w.tiles_per_range < SH) ++w.tiles_per_range;
    if (fit >= 1) {
      const int parts = (SH + w.tiles_per_range - 1) / w.tiles_per_range;
      auto steps = [&](int most_parts) { const int n = parts < most_parts ? parts : most_parts; return n < 1 ? SH : (SH + n - 1) / n; };
      const int full = steps(fit), half = steps(fit / 2);
      const int own = half <= full + 4 ? half : full;
      if (full <= w.tiles_per_range + 2) { w.tiles_per_range = own; w.tiles_per_head = (SH + own - 1) / own * own; }
    }
    w.nranges = (int)(((long)m.heads * w.tiles_per_head + w.tiles_per_range - 1) / w.tiles_per_range);
    // First pass over 256 rows at once or 128 at a time: for the longest heads, and thousands of tokens to a workgroup, operands from LDS cost a
    // little more than a second pass over K through the first-level cache.  Both passes, us, at once and in parts: 256 rows, 288 heads of 4096, 8192,
    // 12000, 20000, 24000, 32768 tokens 194 - 200, 382 - 387, 558 - 566, 932 - 930, 1120 - 1106, 1527 - 1505; 512 heads of 4096 331 - 353; 96 of 12000, 32768
    // 184 - 186, 508 - 508; 512 rows, 512 heads of 2048 322 - 353, 288 of 8192, 20000 704 - 715, 1714 - 1714, 144 of 32768 1393 - 1389; 768 rows, 288 of 20000
    // 2528 - 2550, 96 of 32768 1368 - 1359.  The second pass is ahead throughout, and so is 192 rows at once.
    w.narrow_stats = tall == 256 && m.N >= 24000 && (long)w.tiles_per_range * kScoreTallStep >= 4096;
    if (w.narrow_stats) {
      w.stats_rgroups = (m.R + 127) / 128;
      w.stats_tiles_per_head = (m.N + 31) / 32;
      const long ST = (long)m.heads * w.stats_tiles_per_head;
      w.stats_tiles_per_range = score_tiles_per_range(ST, w.stats_rgroups);
      w.stats_nranges = (int)((ST + w.stats_tiles_per_range - 1) / w.stats_tiles_per_range);
      w.narrow_stats = slots(w.stats_tiles_per_head, w.stats_tiles_per_range) <= most;
    }
  } else {
    w.tiles_per_head = (m.N + 31) / 32;
    int T = score_tiles_per_range((long)m.heads * w.tiles_per_head, w.rgroups);
    w.nslot = slots(w.tiles_per_head, T);                         // (no less for the longer ranges below)
    // Ranges that end with their head, where that makes them at most a round of tiles longer: a range that goes on into the next head loads
    // its queries and fills its pipeline again, 5 us a pass.  128 rows, both passes, before and after: 16 heads of 1300, 2500 and 4100 tokens 35, 38
    // and 42 us, 21, 25 and 29; 120 heads of 1300 and 4100: 43 and 65, 30 and 53; 160 heads would need half as many tiles again and stay.
    // The head is padded with tiles past its tokens, which take no time.
    const int per_head = kNumCU / m.heads;
    if (w.rgroups == 1 && per_head >= 1 && m.dtype == OBF_BF16 && m.d == 128) {
      const int own = ((w.tiles_per_head + per_head - 1) / per_head + 3) / 4 * 4;
      if (own <= T + 4) { T = own; w.tiles_per_head = (w.tiles_per_head + T - 1) / T * T; }
    }
    const long TT = (long)m.heads * w.tiles_per_head;
    w.tiles_per_range = T;
    w.nranges = (int)((TT + T - 1) / T);
  }
  if (!w.narrow_stats) {
    w.stats_rgroups = w.rgroups; w.stats_tiles_per_head = w.tiles_per_head; w.stats_tiles_per_range = w.tiles_per_range; w.stats_nranges = w.nranges;
  }
  if (tall) w.nslot = slots(w.stats_tiles_per_head, w.stats_tiles_per_range);
  else held = w.nchunk > w.nslot ? w.nchunk : w.nslot;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  w.stats_part = take(sizeof(double) * 2 * (size_t)m.heads * held * m.R);
  w.row_lse = take(sizeof(double) * (size_t)m.heads * m.R);
  w.scores = take(sizeof(float) * (size_t)m.heads * m.N);
  // a single group, and the double-precision path, write their sums to the scores
  w.score_part = take(w.rgroups > 1 && !sums_aside && m.dtype == OBF_BF16 && m.d == 128 ? sizeof(float) * (size_t)(w.rgroups - 1) * m.heads * m.N : 0);
  w.head_state = take(sizeof(HeadState) * (size_t)m.heads);
  w.decided = take(sizeof(int32_t) * (size_t)m.heads);
  w.basis = take(sizeof(float) * (size_t)m.heads * m.d * m.d);
  w.gram_part = take(sizeof(float) * (size_t)m.heads * w.nstat * gram_stride(m.d));
  w.mats = take(sizeof(float) * (size_t)m.heads * 3 * m.d * m.d);
  if (w.nslot > held) w.stats_part = w.basis;                    // (basis, gram_part and mats follow each other)
  if (sums_aside) w.score_part = w.basis;                        // (with 128 rows at a time the partials are never there)
  w.delta = take(sizeof(float) * (size_t)m.heads * m.d);
  w.sel_flags = take(sizeof(int32_t) * (size_t)m.heads);
  w.band = take(16 * (size_t)m.heads * kBandCap);
  w.layer_scores = take(sizeof(float) * (size_t)m.L * m.N);
  w.layer_idx = take(sizeof(int32_t) * ((size_t)m.L * (max_budget > 0 ? max_budget : 0) + m.L));
  w.fro_part = take(sizeof(double) * (size_t)m.heads * ((max_budget > 0 ? max_budget : 0) / kGatherRows + 1));
  w.keep_gram = take(max_budget >= kKeepGramMinBudget ? sizeof(double) * kKeepGramSlots * kKeepGramChunks * (size_t)m.d * m.d : 0);
  w.lead_total = off;
  w.rot = take((max_budget < m.d && rank > 0) ? sizeof(float) * (size_t)m.heads * kJacobiSweeps * (m.d - 1) * (m.d / 2) : 0);
  w.inv_norm = take(sizeof(float) * (size_t)m.heads * (max_budget > 0 ? max_budget : 0));
  w.route = take(sizeof(int32_t) * (size_t)m.heads * m.N);
  w.total = off;
  return w;
}

enum Stage {
  ST_SCORE_STATS = 0, ST_SCORE_LSE, ST_SCORE_MASS, ST_SELECT, ST_REFINE, ST_GATHER, ST_KEEP_CERT, ST_KEEP_BASIS, ST_DEL_STATS,
  ST_FINALIZE, ST_BASIS_STATS, ST_COUNT
};

// Brackets one kernel launch with HIP events when profiling of that stage is enabled.
struct ProfScope {
  ProfScope(int stage, hipStream_t st);
  ~ProfScope();
  void* rec;
  hipStream_t st;
};

void set_error(const char* fmt, ...);
obf_status_t check_launch(const char* what);

// ---- device helpers -------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even float -> bf16 bits; NaN stays NaN
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  uint32_t lsb = (u >> 16) & 1u;
  return (uint16_t)((u + 0x7fffu + lsb) >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float load(const float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {
  static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_bits_to_float(*p); }
  static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = float_to_bf16_bits(v); }
};

// ---- stage launchers (each enqueues on `st`, returns OBF_OK or OBF_ERR_HIP) --------------
obf_status_t launch_score_generic(const Dims& m, const Workspace& w, char* ws, const void* K, const void* Q,
                                  float* scores, double* row_lse, hipStream_t st);
bool mfma_score_supported(const Dims& m);
// Both passes with row groups of 192 or 256 rows (the first only where w.narrow_stats does not leave it to the other kernel).  The last group's sums go
// to `scores`, the others' to `part`.
obf_status_t launch_score_tall(const Dims& m, const Workspace& w, double* stats_part, const void* K, const void* Q, float* part, float* scores,
                               double* row_lse, hipStream_t st);
obf_status_t launch_score_mfma(const Dims& m, const Workspace& w, char* ws, const void* K, const void* Q,
                               float* scores, double* row_lse, hipStream_t st);
obf_status_t launch_select(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                           int32_t max_budget, int32_t* idx, int32_t* n_keep, hipStream_t st);
obf_status_t launch_select_refine(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                                  int32_t max_budget, int32_t* idx, int32_t* n_keep, const void* K, const void* Q,
                                  const double* row_lse, hipStream_t st, int32_t* sel_flags = nullptr /*[heads], nullable*/);
// diag[h].select_flags = sel_flags[h] for every head (diagnostics only)
obf_status_t launch_diag_flags(obf_diag_t* diag, const int32_t* sel_flags, int heads, hipStream_t st);
obf_status_t launch_refine(const Dims& m, const Workspace& w, char* ws, const void* K, const void* Q,
                           const float* scores, const double* row_lse, int32_t max_budget, int32_t* idx,
                           const int32_t* n_keep, hipStream_t st);
obf_status_t launch_gather(const Dims& m, const void* K, const void* V, const int32_t* idx, const int32_t* n_keep,
                           int32_t max_budget, void* K_out, void* V_out, hipStream_t st, double* fro_part = nullptr);
// Retained-span basis for the heads with at most head_dim retained rows (the others are left untouched).
obf_status_t launch_keep_basis_small(const Dims& m, const void* V, const float* scores, const int32_t* idx,
                                     const int32_t* n_keep, int32_t max_budget, int32_t rank, HeadState* state,
                                     float* basis, hipStream_t st);
bool del_stats_mfma_supported(const Dims& m);
obf_status_t launch_del_stats_mfma(const Dims& m, const Workspace& w, const void* V, const float* scores,
                                   const int32_t* idx, int32_t max_budget, const HeadState* state,
                                   const int32_t* n_keep /*non-null: do not read the head states*/, float* gram_part,
                                   hipStream_t st, bool few_active = false /*nearly every head is expected to be inactive*/);
obf_status_t launch_del_stats_generic(const Dims& m, const Workspace& w, const void* V, const float* scores, const int32_t* idx,
                                      int32_t max_budget, const HeadState* state,
                                      const int32_t* n_keep /*non-null: do not read the head states*/, float* gram_part, hipStream_t st);
bool keep_cert_supported(const Dims& m, int max_budget);
obf_status_t launch_keep_cert(const Dims& m, const void* Vsrc, int via_idx, const float* scores, const int32_t* idx,
                              const int32_t* n_keep, int32_t max_budget, int32_t rank, HeadState* state,
                              int32_t* decided, hipStream_t st, const double* fro_part = nullptr, bool want_sums = true);
obf_status_t launch_refine_layers(const Dims& m, const void* K, const void* Q, const float* layer_scores,
                                  const double* row_lse, int32_t max_budget, const int32_t* idx_layer,
                                  const int32_t* n_keep_layer, double* part /*[heads][kBandCap]*/, int32_t* idx, int32_t* n_keep, hipStream_t st);
// Layerwise retention rule: TopK_B of the head-summed scores of each layer (with the exact re-decision at the
// threshold), copied to every head of the layer.  budgets_host: per layer (nullable).
obf_status_t launch_select_layerwise(const Dims& m, const Workspace& w, char* ws, const float* scores,
                                     const int32_t* budgets_host, int32_t budget, int32_t max_budget, int32_t* idx,
                                     int32_t* n_keep, const void* K, const void* Q, const double* row_lse,
                                     hipStream_t st);
// Ablation variants of App. D as the kernels see them (obf_variant_t checked and packed).
enum : int { VF_NO_PROJECTION = 1, VF_SUBSPACE_ALL = 2, VF_SUBSPACE_EVR = 4, VF_NO_SCALING = 8, VF_NAIVE = 16, VF_ATTN_INJECT = 32, VF_PER_TOKEN = 64 };
struct Variant {
  int flags = 0;
  float evr_tau = 0.f;
  int subspace_iters = 0;          // > 0: App. H's Gram subspace iteration with this many steps instead of the eigen-decomposition
  bool skips_basis() const { return (flags & (VF_NO_PROJECTION | VF_NAIVE)) != 0; }
};

obf_status_t launch_append_message(int heads, int row_bytes, const void* prev_K, const void* prev_V, const int32_t* prev_len,
                                   int prev_len_all, int prev_stride, const void* keep_K, const void* keep_V,
                                   const int32_t* n_keep, int keep_stride, const void* gen_K, const void* gen_V, int n_gen,
                                   int gen_stride, void* msg_K, void* msg_V, int32_t* msg_len, int msg_stride, hipStream_t st);
// Cache merging (App. E) on selected and gathered rows: routes (route_out nullable) and merged values in V_out.
obf_status_t launch_cache_merge(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores,
                                const int32_t* idx, const int32_t* n_keep, int32_t max_budget, const void* K_out,
                                void* V_out, int32_t* route_out, hipStream_t st);
// The Per-token alternative of App. D after a back-fill that left its subspace in the workspace (flag VF_PER_TOKEN) and
// did not inject: routes as in the cache merging, then one direction per retained slot added to V_out.
obf_status_t launch_per_token_inject(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V,
                                     const float* scores, const int32_t* idx, const int32_t* n_keep, int32_t max_budget,
                                     const void* K_out, void* V_out, int no_scaling, hipStream_t st);
// Per-row int8 / int4 codes of relay rows and back (App. E's stacked quantisation, the reading stated in quant.hip).
obf_status_t launch_quant_rows(const void* X, long n_rows, int d, int dtype, int bits, uint8_t* codes, uint16_t* scale,
                               uint16_t* zero, hipStream_t st);
obf_status_t launch_dequant_rows(const uint8_t* codes, const uint16_t* scale, const uint16_t* zero, long n_rows, int d, int dtype,
                                 int bits, void* X, hipStream_t st);
// Runs `set` (hipFuncSetAttribute calls) once per device: kernel attributes belong to the device that is current when they
// are set.  `seen` and `mu` are the caller's function-local statics; the device's bit is set only after `set` has returned,
// so a second host thread either waits for the mutex or finds the attributes in place.
template <class F>
inline void once_per_device(std::mutex& mu, uint64_t& seen, F set) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { set(); return; }
  std::lock_guard<std::mutex> lock(mu);
  if (seen & (1ull << dev)) return;
  set();
  seen |= 1ull << dev;
}

// idx[i] += offset for every valid (non-negative) entry
obf_status_t launch_idx_offset(int32_t* idx, size_t n, int32_t offset, hipStream_t st);

// The library's own streams: kAuxStreams per host thread and device, default priority, created on first use and kept.
// aux_stream returns nullptr when none is available (creation failed, or the thread is in single-stream mode): the
// launchers then keep everything on the caller's stream.
constexpr int kBatchLanes = 3;                                   // workspace slots of a batch, and samples in flight at a time: with lane 0's
                                                                  // inner fork that makes four streams, one per hardware queue (12 samples of
                                                                  // 165 to 340 tokens, ms a sample: one lane 0.131, two 0.084, three 0.075)
constexpr int kAuxStreams = kBatchLanes;                          // the library's own streams per device and thread
constexpr int kMostLanes = kAuxStreams + 1;                       // where no sample forks
hipStream_t aux_stream(int which /*0 .. kAuxStreams-1*/);
// While on (per host thread), no stream or event is created or used by the library.
void set_single_stream(bool on);
// Makes `waiter` wait for everything queued on `signaller` so far, through event `slot` of the calling thread's pool
// (an event may be recorded again as soon as its wait has been enqueued).  Legal under stream capture.
enum EventSlot { EV_SCORED = 0, EV_BASIS_FORK, EV_BASIS_JOIN, EV_KROWS_FORK, EV_KROWS_JOIN, EV_BATCH_FORK, EV_BATCH_JOIN, EV_COUNT };
obf_status_t stream_after(hipStream_t waiter, hipStream_t signaller, int slot);
// Optional early start of the retained-span bases on `aux` (forked from st), for shapes where they do not depend on
// the gather; *started is then passed on to launch_backfill as Begun::bases, which joins `aux` back.
obf_status_t launch_backfill_basis(const Dims& m, const Workspace& w, char* ws, const void* V, const float* scores,
                                   const int32_t* idx, const int32_t* n_keep, int32_t max_budget, int32_t rank,
                                   hipStream_t st, hipStream_t aux, bool* started);
// Bases, statistics and, with K_out and V_out given, the gathered rows of calls with small budgets in one launch (basis_stats.hip).
bool basis_stats_supported(int32_t max_budget, int32_t rank, int d);
obf_status_t launch_basis_stats(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores,
                                const int32_t* idx, const int32_t* n_keep, int32_t max_budget, int32_t rank, void* K_out /*nullable*/,
                                void* V_out /*nullable*/, hipStream_t st);
// What of the back-fill the caller has already enqueued: nothing; the bases, on `aux`; the bases and the statistics, on `st`.
enum class Begun { nothing, bases, statistics };
// The index lists of a token window, which have to move by `by` once nothing of the call reads them any more; launch_backfill sets `done` if its last
// kernel does that (one launch less: 2 to 3 us).
struct IdxShift { int32_t* idx; int32_t by; bool done; };
obf_status_t launch_backfill(const Dims& m, const Workspace& w, char* ws, const void* V, const float* scores,
                             const int32_t* idx, const int32_t* n_keep, int32_t max_budget, int32_t rank,
                             void* V_out, float* delta_out, obf_diag_t* diag, hipStream_t st, hipStream_t aux /*nullable*/,
                             const double* fro_part = nullptr,
                             Begun begun = Begun::nothing, int32_t min_budget = -1 /*smallest per-head budget if known*/,
                             Variant var = Variant(), IdxShift* shift = nullptr);

// Rank rule with at most kLeadMaxRank directions: everything after the statistics pass (backfill_lead.hip), App. H's fast path included.
constexpr int kLeadMaxRank = 16;
// shift (nullable): its lists move once they have been read.
obf_status_t launch_backfill_lead(const Dims& m, const Workspace& w, char* ws, const float* scores, const int32_t* idx, int32_t max_budget,
                                  int32_t rank, void* V_out /*nullable*/, float* delta_out, obf_diag_t* diag, hipStream_t st, int vflags,
                                  int iters, IdxShift* shift);

}  // namespace obf
