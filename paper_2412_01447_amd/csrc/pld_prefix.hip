// pld_prefix.hip -- prompt lookup's selection, the baseline PLD+ replaces
// (arXiv 2412.01447, Sec. 2; the Fig. 3 caption: prompt lookup proposes the
// candidate span with the longest matching prefix).
//
// For a candidate j (0 <= j <= T-2) the match length is the largest
// m <= max_match with x[j-k] = x[T-1-k] for every k < m (indices j-k >= 0);
// the chosen j* has the largest m, the earliest among equal lengths (prompt
// lookup scans the context from the start and keeps the first match).
//
// Rows of up to 16384 tokens are drafted in one launch (draft_prefix_kernel): the
// search leaves the token row and the list in LDS, where the match lengths are
// taken and the draft is read.  Nothing but the token row is read from memory, and
// what bounds the step is launches: as the separate calls it took three, the
// second and third waiting for a few KB of the one before.  Longer rows, and large
// batches of rows past 8192 tokens, are searched by the find call's launches, and
// one more selects and writes the draft.
#include "pld.h"
#include "pld_device.h"
#include "pld_match.h"

namespace pld {

constexpr int kPrefixThreads = 1024;  // the one-launch form
constexpr int kPrefixWaves = kPrefixThreads / kWave;
constexpr int kPrefixChunk = 16;      // tokens compared per trip to memory (at most)
constexpr int kPrefixChunkLds = 4;    // and to LDS
// Sequences up to which rows of 8193 to 16384 tokens take one launch.  Their tokens
// and list leave a CU room for one block (131 KB of LDS), where the find call's has
// two: past that short lists are faster as find and selection (us per call, the three
// separate calls | one launch | two; 4, 256 and 2048 occurrences each): 1024 x 16384
// 25.9 32.4 55.2 | 24.1 25.4 30.9 | 23.2 27.5 36.0, 2048 x 16384 46.6 58.5 97.9 | 49.3
// 51.9 62.0 | 43.9 52.2 66.9.
constexpr int kDraftOneLaunchB = 1024;

struct PrefixArgs {
    const int32_t *tokens;
    int64_t tok_stride;
    const int32_t *lens;
    const int32_t *cand_pos;
    int64_t cap;
    const int32_t *cand_count;
    int B;
    int max_match;
    float *scores;   // [B][cap] or null
    int32_t *best_pos;
    float *best_score;
    int K;           // 0: no draft
    int32_t *draft;
    int32_t *draft_len;
};

// Compares the kChunk tokens back from x[j-m] with the query's from x[T-1-m],
// advancing m to the first difference or to lim; whether the run goes on.  Loads
// that would reach below x[0] are clamped (their tokens lie past lim <= j + 1).
template <int kChunk, bool kGlobal, class QueryToken>
__device__ __forceinline__ bool match_chunk(const int32_t *x, int64_t j, int lim, QueryToken query,
                                            int &m) {
    int32_t v[kChunk];
    const int64_t at = j - m;
    if (kGlobal && at >= kChunk - 1) {
        typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int g = 0; g < kChunk / 4; ++g) {
            const i32x4 t = *reinterpret_cast<const i32x4 *>(x + at - 4 * g - 3);
            v[4 * g] = t.w;
            v[4 * g + 1] = t.z;
            v[4 * g + 2] = t.y;
            v[4 * g + 3] = t.x;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kChunk; ++k) v[k] = x[max(at - k, (int64_t)0)];
    }
    // The query's tokens are requested together, not each once the one before has
    // matched: four trips to LDS one after the other bound long matches (us per call,
    // one by one | together; every occurrence matching 64 tokens: 64 x 8192, 200 each,
    // in LDS 10.0 | 7.7, 64 x 20000, 500 each, in memory 18.7 | 15.2).
    int32_t q[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) q[k] = query(m + k);
    uint32_t same = 0;
#pragma unroll
    for (int k = 0; k < kChunk; ++k) same |= (v[k] == q[k] ? 1u : 0u) << k;
    const int n = min(__builtin_ctz(~same), lim - m);   // kChunk <= 16: ~same has a bit
    m += n;
    return n == kChunk;
}

// The match length of candidate j (0 <= j <= T-2), kChunk tokens at a time, x in
// global memory (kGlobal) or LDS; `query(k)` gives x[T-1-k] for k < qn, any value past that.  What bounds the
// lanes' scattered reads of memory is the addresses that a CU's load path takes,
// about one a clock: 16 tokens in four 16-byte loads, not sixteen (4 x 100000
// tokens, 2500 occurrences: 40.5 -> 26.5 us per step).  In LDS most candidates
// end within four tokens (us per call, 16 | 8 | 4 at a time: 8 x 4096 tokens, 64
// occurrences each 4.7 | 4.5 | 4.3, 48 x 16384, 256 each 6.6 | 6.2 | 6.0; where every
// one of 200 matches 64 tokens, 64 x 8192, 7.6 | 7.4 | 7.7).
template <int kChunk, bool kGlobal, class QueryToken>
__device__ __forceinline__ int match_length(const int32_t *x, int64_t j, int qn, QueryToken query) {
    // the run can reach back to x[0] and no further than the query suffix
    const int lim = (int)min((int64_t)qn, j + 1);
    int m = 0;
    bool run = true;
    while (run && m < lim) run = match_chunk<kChunk, kGlobal>(x, j, lim, query, m);
    return m;
}

__device__ __forceinline__ uint64_t prefix_key(int m, int64_t j) {
    return ((uint64_t)(uint32_t)m << 32) | (uint64_t)(0xffffffffu - (uint32_t)j);
}

// The best key of a block of kWaves waves as the ranking's (score, position) key,
// in every thread of its first wave; `s_key` is one word per wave.
template <int kWaves>
__device__ __forceinline__ uint64_t block_choice(uint64_t best, uint64_t *s_key) {
    best = wave_max_u64(best);
    if (lane_id() == 0) s_key[threadIdx.x / kWave] = best;
    lds_barrier();
    if (threadIdx.x >= kWave) return 0ull;
    const uint64_t k = wave_max_u64(lane_id() < kWaves ? s_key[lane_id()] : 0ull);
    return k ? rank_key((float)(uint32_t)(k >> 32), (int32_t)(0xffffffffu - (uint32_t)k)) : 0ull;
}

// One block per sequence over a list in memory.  The query suffix is staged in
// LDS; a lane takes a candidate, kChunk tokens at a time.  launch_select_prefix
// picks the form.
template <int kThreads, int kChunk>
__global__ __launch_bounds__(kThreads) void select_prefix_kernel(PrefixArgs a) {
    static_assert(kChunk <= kPrefixChunk, "s_q is read up to kChunk - 1 past the suffix");
    __shared__ int32_t s_q[PLD_MAX_MATCH + kPrefixChunk];   // x[T-1-k]
    __shared__ uint64_t s_key[kThreads / kWave];
    const int b = blockIdx.x;
    const int32_t *x = a.tokens + (int64_t)b * a.tok_stride;
    const int64_t T = a.lens[b];
    int64_t C = a.cand_count[b];
    if (C < 0 || C > a.cap) C = 0;
    const bool seq_ok = T >= 2 && T <= a.tok_stride;   // block-uniform
    const int qn = seq_ok ? (int)min((int64_t)a.max_match, T) : 0;
    for (int k = threadIdx.x; k < qn; k += kThreads) s_q[k] = x[T - 1 - k];
    __syncthreads();

    const int32_t *pos = a.cand_pos + (int64_t)b * a.cap;
    uint64_t best = 0;
    for (int64_t c = threadIdx.x; c < (seq_ok ? C : 0); c += kThreads) {
        const int64_t j = pos[c];
        float s = NAN;
        if (j >= 0 && j <= T - 2) {
            const int m = match_length<kChunk, true>(x, j, qn, [&](int k) { return s_q[k]; });
            s = (float)m;
            const uint64_t key = prefix_key(m, j);
            best = key > best ? key : best;
        }
        if (a.scores) a.scores[(int64_t)b * a.cap + c] = s;
    }
    best = block_choice<kThreads / kWave>(best, s_key);
    if (threadIdx.x < kWave)
        write_choice_draft(best, T, seq_ok, x, a.K, a.best_pos + b, a.best_score + b,
                           a.K ? a.draft + (int64_t)b * a.K : nullptr,
                           a.K ? a.draft_len + b : nullptr);
}

struct DraftPrefixArgs {
    PrefixArgs p;        // cand_pos and cand_count unused
    int nmin, nmax;
    int32_t *cand_pos;
    int32_t *cand_count;
    int32_t *ngram_used;
};

// One block per sequence, tok_stride <= kPasses * kFindFusedMax: the search of the
// one-block find, its list in LDS as well, then a lane per candidate.  With one pass
// two blocks share a CU (66 KB of LDS each; up to 64 registers, eight waves per
// SIMD), which is what bounds large batches (us per call, the three separate calls |
// one block per CU | two; 128 occurrences or fewer): 512 x 8192 14.5 | 9.4 | 7.7, 4096 x
// 8192 64.0 | 57.3 | 39.8, 4096 x 1024 34.6 | 36.2 | 25.8, 16384 x 512 115 | 134 | 91.
template <int kPasses>
__global__ __launch_bounds__(kPrefixThreads, kPasses == 1 ? 8 : 4) void draft_prefix_kernel(DraftPrefixArgs d) {
    static_assert(kPrefixWaves == kFindWavesFused, "the search takes the whole block");
    constexpr int G = kPasses * kFindFusedMax / kPrefixThreads;
    __shared__ __align__(16) int32_t s_x[kPasses * kFindFusedMax];
    __shared__ int32_t s_list[kPasses * kFindFusedMax];
    __shared__ int s_lvl[kPrefixWaves][kMaxNgram];
    __shared__ uint64_t s_key[kPrefixWaves];
    const PrefixArgs &a = d.p;
    const int b = blockIdx.x;
    const int32_t *x = a.tokens + (int64_t)b * a.tok_stride;
    // the whole token row is requested with the length, not after it
    const int64_t T = a.lens[b];
    if (((uintptr_t)x & 15) == 0 && (a.tok_stride & 3) == 0)
        copy_to_lds(reinterpret_cast<const uint4 *>(x), reinterpret_cast<uint4 *>(s_x),
                    (int)(a.tok_stride / 4));
    else
        stage_tokens(x, 0, a.tok_stride, s_x);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const bool tok_ok = T >= 1 && T <= a.tok_stride;   // block-uniform
    int n_used = -1, total = 0;
    if (tok_ok)
        n_used = block_search<kPrefixWaves, G>(s_x, T, d.nmin, d.nmax, s_lvl, s_list, total);
    lds_barrier();   // the list is complete
    if (threadIdx.x == 0) {
        d.cand_count[b] = total;
        d.ngram_used[b] = n_used;
    }
    // every listed position lies in [1, T-2]
    const int qn = tok_ok ? (int)min((int64_t)a.max_match, T) : 0;
    uint64_t best = 0;
    for (int c = threadIdx.x; c < total; c += kPrefixThreads) {
        const int32_t j = s_list[c];
        d.cand_pos[(int64_t)b * a.cap + c] = j;
        const int m = match_length<kPrefixChunkLds, false>(
            s_x, j, qn, [&](int k) { return s_x[max((int)T - 1 - k, 0)]; });
        const uint64_t key = prefix_key(m, j);
        best = key > best ? key : best;
        if (a.scores) a.scores[(int64_t)b * a.cap + c] = (float)m;
    }
    best = block_choice<kPrefixWaves>(best, s_key);
    if (threadIdx.x < kWave)
        write_choice_draft(best, T, tok_ok, s_x, a.K, a.best_pos + b, a.best_score + b,
                           a.draft + (int64_t)b * a.K, a.draft_len + b);
}

// Up to 256 sequences there is a CU for each, and 1024 threads make the few thousand
// candidates of a long context few dependent rounds (position, tokens); up to 512,
// two blocks of 512 threads share one.  Past that what bounds the call is how many
// short lists a CU takes at once: 256 threads, whose 8-token chunks need half the
// registers of 16 (28, not 60).  Measured (us per call, 1024 threads | 512 | 256 of
// 16-token chunks | 256 of 8): 256 x 16384 tokens, 256 occurrences each 5.0 | 5.0 | 5.5 |
// 5.2, 2048 each 7.1 | 8.0 | 11.0 | 10.5; 512 x 4096, 4 each 4.2 | 3.7 | 4.2 | 3.7, 512 x
// 16384, 2048 each 9.6 | 10.1 | 12.3 | 11.8; 2048 x 4096, 64 each 13.3 | 8.8 | 6.4 | 6.0,
// 4096 x 4096, 4 each 18.1 | 11.1 | 6.7 | 6.3, 65535 x 128, 8 each 330 | 189 | 79 | 71.
static void launch_select_prefix(const PrefixArgs &a, hipStream_t s) {
    const dim3 grid((unsigned)a.B);
    if (a.B <= 256)
        hipLaunchKernelGGL((select_prefix_kernel<1024, 16>), grid, dim3(1024), 0, s, a);
    else if (a.B <= 512)
        hipLaunchKernelGGL((select_prefix_kernel<512, 16>), grid, dim3(512), 0, s, a);
    else
        hipLaunchKernelGGL((select_prefix_kernel<256, 8>), grid, dim3(256), 0, s, a);
}

}  // namespace pld

using namespace pld;

extern "C" int pld_select_prefix(const int32_t *tokens, int64_t tok_stride, const int32_t *lens,
                                 const int32_t *cand_pos, int64_t cap, const int32_t *cand_count,
                                 int B, int max_match, float *scores, int32_t *best_pos,
                                 float *best_score, void *stream) {
    if (!tokens || !lens || !cand_pos || !cand_count || !best_pos || !best_score)
        return PLD_ERR_INVALID;
    if (B < 1 || B > 65535 || tok_stride < 1 || tok_stride > kMaxTokStride || cap < 1)
        return PLD_ERR_INVALID;
    if (max_match < 1 || max_match > PLD_MAX_MATCH) return PLD_ERR_INVALID;
    PrefixArgs a{tokens, tok_stride, lens, cand_pos, cap, cand_count, B, max_match,
                 scores,  best_pos,   best_score, 0, nullptr, nullptr};
    launch_select_prefix(a, (hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? PLD_OK : PLD_ERR_LAUNCH;
}

extern "C" int pld_draft_prefix(const int32_t *tokens, int64_t tok_stride, const int32_t *lens,
                                int B, int ngram_min, int ngram_max, int max_match, int K,
                                int32_t *cand_pos, int64_t cap, int32_t *cand_count,
                                int32_t *ngram_used, float *scores, int32_t *best_pos,
                                float *best_score, int32_t *draft, int32_t *draft_len,
                                void *scratch, size_t scratch_bytes, void *stream) {
    if (!tokens || !lens || !cand_pos || !cand_count || !ngram_used || !best_pos || !best_score ||
        !draft || !draft_len)
        return PLD_ERR_INVALID;
    if (B < 1 || B > 65535 || tok_stride < 1 || tok_stride > kMaxTokStride) return PLD_ERR_INVALID;
    if (ngram_min < 1 || ngram_max < ngram_min || ngram_max > PLD_MAX_NGRAM) return PLD_ERR_INVALID;
    if (cap < tok_stride || K < 1) return PLD_ERR_INVALID;
    if (max_match < 1 || max_match > PLD_MAX_MATCH) return PLD_ERR_INVALID;
    if (((int64_t)B * K + 255) / 256 > 0x7fffffff) return PLD_ERR_INVALID;   // as pld_emit_draft
    const PrefixArgs a{tokens, tok_stride, lens, cand_pos, cap, cand_count, B, max_match,
                       scores,  best_pos,   best_score, K, draft, draft_len};
    const hipStream_t s = (hipStream_t)stream;
    const dim3 grid((unsigned)B), threads(kPrefixThreads);
    if (tok_stride <= kFindFusedMax ||
        (tok_stride <= kFindFusedPasses * kFindFusedMax && B <= kDraftOneLaunchB)) {
        const DraftPrefixArgs d{a, ngram_min, ngram_max, cand_pos, cand_count, ngram_used};
        if (tok_stride <= kFindFusedMax)
            hipLaunchKernelGGL(draft_prefix_kernel<1>, grid, threads, 0, s, d);
        else
            hipLaunchKernelGGL(draft_prefix_kernel<kFindFusedPasses>, grid, threads, 0, s, d);
    } else {
        const int rc = pld_find_candidates(tokens, tok_stride, lens, B, ngram_min, ngram_max,
                                           cand_pos, cap, cand_count, ngram_used, scratch,
                                           scratch_bytes, stream);
        if (rc != PLD_OK) return rc;
        launch_select_prefix(a, s);
    }
    return hipGetLastError() == hipSuccess ? PLD_OK : PLD_ERR_LAUNCH;
}
