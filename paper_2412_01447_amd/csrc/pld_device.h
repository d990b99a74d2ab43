// pld_device.h -- device helpers shared by the PLD+ kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "this library is written for gfx950 (MI355X) only"
#endif

namespace pld {

constexpr int kWave = 64;
constexpr int kMaxNgram = 8;                   // equals PLD_MAX_NGRAM
constexpr int64_t kMaxTokStride = 1ll << 30;   // positions are stored as int32

// Tiling of the occurrence search.
constexpr int kFindTile = 2048;          // positions per block, multi-block find
constexpr int kFindWavesTiled = 4;       // 256 threads, 512 positions per wave
constexpr int kFindWavesFused = 16;      // 1024 threads, one block per sequence
constexpr int kFindFusedMax = kFindWavesFused * 512;  // tok_stride <= 8192: fused path
#ifndef PLD_FIND_FUSED_PASSES
#define PLD_FIND_FUSED_PASSES 2
#endif
constexpr int kFindFusedPasses = PLD_FIND_FUSED_PASSES;   // one-block search: tok_stride <= 16384

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Whether the byte ranges [p, p + np) and [q, q + nq) share a byte.
inline bool ranges_overlap(const void *p, size_t np, const void *q, size_t nq) {
    const uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return a < b + nq && b < a + np;
}

// Blocks of `kernel` that fit on the current device at once (CUs x resident
// blocks per CU): the grid of the persistent kernels, whose equal contiguous
// work ranges then finish in a single round.  Kept per device, kernel and
// dynamic LDS size in a table whose slots are taken over by the latest asker, so
// that a program of many batch sizes and widths does not run out of room and query
// the occupancy on every call.
inline int resident_blocks(const void *kernel, int threads, size_t dyn_lds) {
    struct Entry {
        int dev;
        const void *k;
        size_t lds;
        int blocks;
    };
    constexpr size_t kSlots = 1024;
    static std::mutex mu;
    static Entry table[kSlots];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    // kernel handles lie 8 bytes or more apart, the LDS sizes asked for as well
    Entry &e = table[((uintptr_t)kernel / 8 * 67 + dyn_lds / 8 + (size_t)dev * 131) % kSlots];
    {
        std::lock_guard<std::mutex> g(mu);
        if (e.k == kernel && e.lds == dyn_lds && e.dev == dev) return e.blocks;
    }
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, dyn_lds) != hipSuccess ||
        per < 1)
        per = 1;
    const int blocks = cus * per;
    std::lock_guard<std::mutex> g(mu);
    e = Entry{dev, kernel, dyn_lds, blocks};
    return blocks;
}

// Tiles per sequence up to which each compaction block sums the per-tile
// counts itself (a few KB per block); past it a scan launch gives every tile
// its offset, so the work grows with the tiles, not with their square.
constexpr int kFindScanTiles = 256;

// Scratch of the multi-block find: per-tile occurrence counts of every n;
// past kFindScanTiles tiles also the per-tile offsets of the chosen n and
// each sequence's (n, count).
inline size_t find_scratch_bytes(int B, int64_t tok_stride) {
    if (tok_stride <= kFindFusedPasses * kFindFusedMax) return 0;   // the one-block search
    const int64_t ntiles = (tok_stride + kFindTile - 1) / kFindTile;
    size_t bytes = align_up((size_t)B * (size_t)ntiles * 8 * sizeof(int32_t), 256);
    if (ntiles > kFindScanTiles)
        bytes += align_up((size_t)B * (size_t)ntiles * sizeof(int32_t), 256) +
                 align_up((size_t)B * 2 * sizeof(int32_t), 256);
    return bytes;
}
// Workspace of the ranking and verification calls: 64-bit keys that must be
// zero when a call starts and that the call leaves zero.  The ranking keys of
// a sequence are spread over kKeySlots slots (a block folds into slot
// blockIdx % kKeySlots), so that few atomics ever queue on one address.
constexpr int kKeySlots = 16;
inline size_t rank_ws_bytes(int B) {
    return align_up((size_t)B * kKeySlots * sizeof(uint64_t), 256);
}
inline size_t verify_ws_bytes(int B, int K) {
    return align_up((size_t)B * ((size_t)K + 1) * sizeof(uint64_t), 256);
}

// ---------------------------------------------------------------- keys
// Order-preserving map of a float to uint32 (larger float -> larger key);
// -0 is folded into +0 first so that the two compare equal.
__device__ __forceinline__ uint32_t ord_f32(float f) {
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord_f32(uint32_t o) {
    uint32_t u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
    return __uint_as_float(u);
}

// Ranking key: highest score first, then the most recent position (j >= 1,
// so 0 means "no eligible candidate").
__device__ __forceinline__ uint64_t rank_key(float s, int32_t j) {
    return ((uint64_t)ord_f32(s) << 32) | (uint32_t)j;
}
// Argmax key over a vocabulary row: highest value first, then the lowest id.
__device__ __forceinline__ uint64_t argmax_key(float v, uint32_t idx) {
    return ((uint64_t)ord_f32(v) << 32) | (uint64_t)(0xffffffffu - idx);
}
__device__ __forceinline__ uint32_t argmax_key_index(uint64_t k) {
    return 0xffffffffu - (uint32_t)(k & 0xffffffffu);
}

// ------------------------------------------------------- wave reductions
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Wave reductions use DPP lane moves -- quad permutes, the half-row and row
// mirrors, and the row broadcasts of lanes 15 and 31 -- a few cycles each,
// where a shuffle goes through the LDS crossbar.  The total lands in lane 63
// and is read back as a scalar, so every lane gets the same bits, and the
// association depends only on the lane layout, never on the data.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_move(int v) {   // lanes the move does not reach get 0
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xf, false);
}
constexpr int kDppQuadSwap1 = 0xb1;   // quad_perm [1,0,3,2]
constexpr int kDppQuadSwap2 = 0x4e;   // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;
constexpr int kDppBcast15 = 0x142;    // lane 15 of a row into the next row (rows 1, 3)
constexpr int kDppBcast31 = 0x143;    // lane 31 into rows 2 and 3
constexpr int kDppShr1 = 0x111;       // row_shr:1 (+1, +3, +7 likewise)

__device__ __forceinline__ int wave_sum_i32(int v) {
    v += dpp_move<kDppQuadSwap1, 0xf>(v);
    v += dpp_move<kDppQuadSwap2, 0xf>(v);
    v += dpp_move<kDppHalfMirror, 0xf>(v);
    v += dpp_move<kDppMirror, 0xf>(v);
    v += dpp_move<kDppBcast15, 0xa>(v);
    v += dpp_move<kDppBcast31, 0xc>(v);
    return __builtin_amdgcn_readlane(v, 63);
}

// Maximum over the lanes of non-negative values (a move's unreached lanes
// read 0, which no lane's value is below).
__device__ __forceinline__ int wave_max_nonneg_i32(int v) {
    v = max(v, dpp_move<kDppQuadSwap1, 0xf>(v));
    v = max(v, dpp_move<kDppQuadSwap2, 0xf>(v));
    v = max(v, dpp_move<kDppHalfMirror, 0xf>(v));
    v = max(v, dpp_move<kDppMirror, 0xf>(v));
    v = max(v, dpp_move<kDppBcast15, 0xa>(v));
    v = max(v, dpp_move<kDppBcast31, 0xc>(v));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ float wave_sum_f32(float v) {
    v += __int_as_float(dpp_move<kDppQuadSwap1, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppQuadSwap2, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppHalfMirror, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppMirror, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppBcast15, 0xa>(__float_as_int(v)));
    v += __int_as_float(dpp_move<kDppBcast31, 0xc>(__float_as_int(v)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint64_t dpp_max_step(uint64_t v) {
    const uint32_t lo = (uint32_t)dpp_move<kCtrl, kRowMask>((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)dpp_move<kCtrl, kRowMask>((int)(uint32_t)(v >> 32));
    const uint64_t o = ((uint64_t)hi << 32) | lo;
    return o > v ? o : v;
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    v = dpp_max_step<kDppQuadSwap1, 0xf>(v);
    v = dpp_max_step<kDppQuadSwap2, 0xf>(v);
    v = dpp_max_step<kDppHalfMirror, 0xf>(v);
    v = dpp_max_step<kDppMirror, 0xf>(v);
    v = dpp_max_step<kDppBcast15, 0xa>(v);
    v = dpp_max_step<kDppBcast31, 0xc>(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// A DPP move whose unreached lanes get `fill` (the identity of the caller's
// operation) instead of 0.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_move_f(float v, float fill) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(fill), __float_as_int(v),
                                                      kCtrl, kRowMask, 0xf, false));
}

__device__ __forceinline__ float wave_max_f32(float v) {
    v = fmaxf(v, dpp_move_f<kDppQuadSwap1, 0xf>(v, -INFINITY));
    v = fmaxf(v, dpp_move_f<kDppQuadSwap2, 0xf>(v, -INFINITY));
    v = fmaxf(v, dpp_move_f<kDppHalfMirror, 0xf>(v, -INFINITY));
    v = fmaxf(v, dpp_move_f<kDppMirror, 0xf>(v, -INFINITY));
    v = fmaxf(v, dpp_move_f<kDppBcast15, 0xa>(v, -INFINITY));
    v = fmaxf(v, dpp_move_f<kDppBcast31, 0xc>(v, -INFINITY));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Inclusive prefix sum of floats over the lanes, in a fixed association.
__device__ __forceinline__ float wave_incl_scan_f32(float x) {
    x += dpp_move_f<kDppShr1, 0xf>(x, 0.f);
    x += dpp_move_f<kDppShr1 + 1, 0xf>(x, 0.f);
    x += dpp_move_f<kDppShr1 + 3, 0xf>(x, 0.f);
    x += dpp_move_f<kDppShr1 + 7, 0xf>(x, 0.f);
    x += dpp_move_f<kDppBcast15, 0xa>(x, 0.f);
    x += dpp_move_f<kDppBcast31, 0xc>(x, 0.f);
    return x;
}

// Exclusive prefix sum over the lanes (shifts by 1, 2, 4, 8 within each row
// of 16, then the row broadcasts); `total` gets the wave's sum.
__device__ __forceinline__ int wave_excl_scan(int v, int &total) {
    int x = v;
    x += dpp_move<kDppShr1, 0xf>(x);
    x += dpp_move<kDppShr1 + 1, 0xf>(x);
    x += dpp_move<kDppShr1 + 3, 0xf>(x);
    x += dpp_move<kDppShr1 + 7, 0xf>(x);
    x += dpp_move<kDppBcast15, 0xa>(x);
    x += dpp_move<kDppBcast31, 0xc>(x);
    total = __builtin_amdgcn_readlane(x, 63);
    return x - v;
}

__device__ __forceinline__ uint64_t lanemask_lt() {
    int l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// Loads of data read exactly once per call (logits rows, candidate hidden
// rows): the nontemporal hint streams them past the caches, which measurably
// raises the HBM read rate on gfx950.  (The attention gathers are not in this
// class: nearby candidates share 128-byte lines of weights.)
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const uint4 *p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// A block barrier that orders LDS accesses alone: the wave waits for its own
// LDS operations, not, as __syncthreads does, for its global stores and copies
// into LDS still on their way (about a microsecond where a list or scores have
// just been stored).  What a copy_to_lds brings is not covered.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Copies n 16-byte chunks from global memory straight into LDS (block-wide)
// with global_load_lds_dwordx4: no registers are held, the copy runs while the
// block does other work, and it is complete after the block's next
// `s_waitcnt vmcnt(0)` + barrier.  Lane l of a wave lands at the wave's LDS
// base + 16 l, so the chunks land in order.
__device__ __forceinline__ void copy_to_lds(const uint4 *g, uint4 *lds, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int i0 = (int)(threadIdx.x - lane); i0 < n; i0 += (int)blockDim.x) {
        if (i0 + lane < n)
            __builtin_amdgcn_global_load_lds(
                (const void *)(g + i0 + lane),
                (__attribute__((address_space(3))) void *)(lds + i0), 16, 0, 0);
    }
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// ------------------------------------------------------- cosine pieces
// Dot products and squared norms of bf16 rows against the bf16 query row in
// LDS, with the gfx950 bf16 dot instruction (v_dot2c_f32_bf16: two bf16
// products added to an fp32 accumulator).  Lane l owns the 8-element chunks
// l, l+64, l+128, ... of a row, in that order; pair p of a chunk accumulates
// into acc[p]; the four accumulators are added as (a0+a1)+(a2+a3) and then
// summed across the wave by a butterfly.  The order depends only on d, so a
// row gives the same bits whichever slot, wave, block or kernel scores it,
// and a row equal to the query gives a dot product equal to both norms.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                           __builtin_bit_cast(bf16x2_t, b), c, false);
}

__device__ __forceinline__ void accum_chunk(const uint4 &h, const uint4 &q, float (&ad)[4],
                                            float (&an)[4]) {
    ad[0] = dot2(h.x, q.x, ad[0]);
    ad[1] = dot2(h.y, q.y, ad[1]);
    ad[2] = dot2(h.z, q.z, ad[2]);
    ad[3] = dot2(h.w, q.w, ad[3]);
    an[0] = dot2(h.x, h.x, an[0]);
    an[1] = dot2(h.y, h.y, an[1]);
    an[2] = dot2(h.z, h.z, an[2]);
    an[3] = dot2(h.w, h.w, an[3]);
}

__device__ __forceinline__ void finish_row(const float (&ad)[4], const float (&an)[4], float &dot,
                                           float &nrm) {
    dot = wave_sum_f32((ad[0] + ad[1]) + (ad[2] + ad[3]));
    nrm = wave_sum_f32((an[0] + an[1]) + (an[2] + an[3]));
}

// One candidate row of any width: up to 16 chunks per lane requested at once.
__device__ __forceinline__ void row_dot(const uint4 *row, const uint4 *q, int nch, float &dot,
                                        float &nrm) {
    constexpr int U = 16;
    const int lane = lane_id();
    float ad[4] = {0.f, 0.f, 0.f, 0.f}, an[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = lane; c0 < nch; c0 += kWave * U) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ch = c0 + u * kWave;
            if (ch < nch) v[u] = ld_stream(row + ch);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ch = c0 + u * kWave;
            if (ch < nch) accum_chunk(v[u], q[ch], ad, an);
        }
    }
    finish_row(ad, an, dot, nrm);
}

// The query row's squared norm from its LDS copy, in row_dot's order (lane l:
// chunks l, l+64, ..., pair p into acc[p]) with one chunk in hand at a time,
// so that it costs few registers; the same bits as row_dot(q, q).
__device__ __forceinline__ float query_norm(const uint4 *q, int nch) {
    float ad[4] = {0.f, 0.f, 0.f, 0.f}, an[4] = {0.f, 0.f, 0.f, 0.f};
    for (int ch = lane_id(); ch < nch; ch += kWave) {
        const uint4 v = q[ch];
        accum_chunk(v, v, ad, an);
    }
    float dot, nrm;
    finish_row(ad, an, dot, nrm);
    return nrm;
}

// Candidate rows streamed through a two-deep pipeline of pieces: the wave keeps
// the loads of the next piece in flight while it reduces the current one, so
// its memory queue never drains the way a load-all-then-wait round does.  Rows
// have up to 64 kLoads chunks of 8 bf16, kLoads 16-byte loads per lane of which
// only the last can be short (masked by chunk).  A piece is kRows whole rows
// (kRows > 0) or half a row (kRows = 0).  with_row_form picks the form.
// The accumulation order is row_dot's (lane l visits its chunks l, l+64,
// l+128, ... in order, pair p of a chunk into acc[p]), so a row gives the same
// bits here as through row_dot.
// `row(k)` gives the k-th row (k < n) of this wave, or null for an unusable
// one (its results are reported as not valid), once per row in whole-row pieces;
// `begin()` runs once the first two pieces are requested (the query's norm is taken
// there, under their latency); `done(k, valid, dot, nrm)` runs in every lane when
// row k is complete, in order of k.
template <int kRows, int kLoads, class RowPtr, class Begin, class Done>
__device__ __forceinline__ void stream_rows(int n, int nch, RowPtr row, const uint4 *q,
                                            Begin begin, Done done) {
    const int lane = lane_id();
    auto has = [&](int u) { return u < kLoads - 1 || u * kWave + lane < nch; };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};
    if constexpr (kRows > 0) {
        uint4 buf[2][kRows][kLoads];
        bool have[2][kRows];
        auto issue = [&](auto slot, int k0) {
            constexpr int sl = decltype(slot)::value;
#pragma unroll
            for (int g = 0; g < kRows; ++g) {
                const uint4 *r = k0 + g < n ? row(k0 + g) : nullptr;
                have[sl][g] = r != nullptr;
                if (r) {
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        if (has(u)) buf[sl][g][u] = ld_stream(r + lane + u * kWave);
                }
            }
        };
        auto consume = [&](auto slot, int k0) {
            constexpr int sl = decltype(slot)::value;
            float dot[kRows], nrm[kRows];
#pragma unroll
            for (int g = 0; g < kRows; ++g) {
                float ad[4] = {0.f, 0.f, 0.f, 0.f}, an[4] = {0.f, 0.f, 0.f, 0.f};
                if (have[sl][g]) {
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        if (has(u)) accum_chunk(buf[sl][g][u], q[lane + u * kWave], ad, an);
                }
                // (no sums over the lanes for the rows that a short piece lacks)
                if (kRows == 1 || k0 + g < n) finish_row(ad, an, dot[g], nrm[g]);
            }
#pragma unroll
            for (int g = 0; g < kRows; ++g)
                if (k0 + g < n) done(k0 + g, have[sl][g], dot[g], nrm[g]);
        };
        issue(first, 0);
        issue(second, kRows);
        begin();
        for (int k = 0; k < n; k += 2 * kRows) {
            consume(first, k);
            issue(first, k + 2 * kRows);
            if (k + kRows < n) {
                consume(second, k + kRows);
                issue(second, k + 3 * kRows);
            }
        }
    } else {
        constexpr int kHalf = (kLoads + 1) / 2;      // loads of piece 0
        uint4 buf[2][kHalf];
        float ad[4] = {0.f, 0.f, 0.f, 0.f}, an[4] = {0.f, 0.f, 0.f, 0.f};
        auto issue = [&](auto piece, int k) {
            constexpr int p = decltype(piece)::value;
            const uint4 *r = row(k);
            if (r) {
#pragma unroll
                for (int u = 0; u < kHalf && p * kHalf + u < kLoads; ++u)
                    if (has(p * kHalf + u))
                        buf[p][u] = ld_stream(r + lane + (p * kHalf + u) * kWave);
            }
        };
        auto consume = [&](auto piece, int k) {
            constexpr int p = decltype(piece)::value;
            const bool ok = row(k) != nullptr;
            if (p == 0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) ad[i] = an[i] = 0.f;
            }
            if (ok) {
#pragma unroll
                for (int u = 0; u < kHalf && p * kHalf + u < kLoads; ++u)
                    if (has(p * kHalf + u))
                        accum_chunk(buf[p][u], q[lane + (p * kHalf + u) * kWave], ad, an);
            }
            if (p == 1) {
                float dot, nrm;
                finish_row(ad, an, dot, nrm);
                done(k, ok, dot, nrm);
            }
        };
        if (n > 0) {
            issue(first, 0);
            issue(second, 0);
        }
        begin();
        for (int k = 0; k < n; ++k) {
            consume(first, k);
            if (k + 1 < n) issue(first, k + 1);
            consume(second, k);
            if (k + 1 < n) issue(second, k + 1);
        }
    }
}

// Calls f(integral_constant<kRows>, integral_constant<kLoads>) with the form
// in which rows of width d stream, or (0, 0) past 8192 (row_dot, one row at a
// time).  A piece holds a few narrow rows, four to eight loads per lane, else a whole
// row, up to twelve loads: past that two pieces no longer fit the 128 registers
// that keep four waves per SIMD (two 8-wave blocks per CU) in the drafting kernels,
// and half a row is a piece.  The ranking kernels need more beside the rows: with
// eleven and twelve loads three waves per SIMD are left (both rankings) or with
// twelve alone (hidden states), which costs them less than the waits of the form
// before (us per call, all loads of a row, then a wait | whole rows | half rows; 32 x
// 16384 tokens, 360 occurrences each: d = 5632 29.0 | 26.9 | 25.8, with 16 heads 31.6 |
// 31.1 | 29.5, with 64 39.7 | 37.8 | 38.1; 6144 31.3 | 29.0 | 28.2, 34.7 | 32.4 | 32.5,
// 41.9 | 39.2 | 40.1).  Measured as one-call
// drafting of 8 x 65536 tokens with 1600 occurrences each (us per step, whole
// rows | half rows | all loads of one to four rows, then a wait): d = 512
// 23.0 | - | 24.5, 1024 25.0 | - | 25.5, 2048 28.9 | - | 28.8, 3584 35.1 | - |
// 35.6, 4096 37.2 | 40.4 | -, 5120 41.6 | 43.6 | 43.5, 6144 47.5 | 47.9 | 48.3,
// 7168 51.3 | 53.2 | 53.0, 8192 55.8 | 56.0 | -; but 44 x 16917 tokens with few
// occurrences, d = 7168, take 39.2 | 35.6 | 35.6, the blocks no longer resident
// together.  Few rows to a piece keep the rows of a short list from waiting for each
// other, more rows keep a long one's loads in flight.  us per call: d = 512 in one block
// per sequence, 8 x 2048 tokens with 16, 64 and 512 occurrences each, load-all-then-wait
// 6.7 8.5 32.1 | eight rows 8.3 9.8 32.8 | four 5.8 7.8 29.1 | two 5.4 7.5 28.8, and the
// ranking call alone, 8 x 8192 with 512 each, 9.4 | 11.8 | 9.3 | 9.6; d = 1024 6.9 8.9 36.0 |
// four 6.0 8.4 33.2 | three 5.8 8.4 33.0 | two 5.6 8.1 32.8, both rankings with 16 heads,
// 256 x 1024 with 128 each, 22.7 | 23.4 | 22.5 | 24.1.
template <class F>
inline void with_row_form(int d, F f) {
    using std::integral_constant;
#define PLD_ROW_FORM(rows, loads) \
    return f(integral_constant<int, rows>{}, integral_constant<int, loads>{})
    switch ((d + 511) / 512) {   // 16-byte loads per lane and row
    case 1: PLD_ROW_FORM(4, 1);
    case 2: PLD_ROW_FORM(3, 2);
    case 3: PLD_ROW_FORM(2, 3);
    case 4: PLD_ROW_FORM(2, 4);
    case 5: PLD_ROW_FORM(1, 5);
    case 6: PLD_ROW_FORM(1, 6);
    case 7: PLD_ROW_FORM(1, 7);
    case 8: PLD_ROW_FORM(1, 8);
    case 9: PLD_ROW_FORM(1, 9);
    case 10: PLD_ROW_FORM(1, 10);
    case 11: PLD_ROW_FORM(1, 11);
    case 12: PLD_ROW_FORM(1, 12);
    case 13: PLD_ROW_FORM(0, 13);
    case 14: PLD_ROW_FORM(0, 14);
    case 15: PLD_ROW_FORM(0, 15);
    case 16: PLD_ROW_FORM(0, 16);
    default: PLD_ROW_FORM(0, 0);
    }
#undef PLD_ROW_FORM
}

// Aggregated attention of one candidate (Eq. 3 / Sec. 7.1), gathered by a
// group of kGatherLanes consecutive lanes: lane t of the group reads the
// weights A[r][j-1] of rows r = t, t+8, t+16, ... (col = &A[0][j-1], rows ar
// apart), up to 8 of them requested at once, and sums them in that order in
// fp32 (or takes their maximum); the group's eight partials are then combined
// by DPP moves inside the group (lane xor 1, xor 2, then the half-row mirror),
// which leaves the same bits in every lane of the group.  A candidate's R loads
// are thus one trip to memory for R <= 64.  Plain (cached) loads: candidates
// a few positions apart read the same 128-byte lines, and a line kept in L2
// serves the second one.  Call with the whole wave converged; `active` masks
// the loads of lanes without a candidate.
constexpr int kGatherLanes = 8;
__device__ __forceinline__ float attn_gather_group(const float *col, int64_t ar, int R, bool sum,
                                                   bool active) {
    const int t = lane_id() & (kGatherLanes - 1);
    const float none = sum ? 0.f : -INFINITY;
    float acc = none;
    for (int r0 = 0; r0 < R; r0 += 8 * kGatherLanes) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int r = r0 + u * kGatherLanes + t;
            v[u] = (active && r < R) ? col[(int64_t)r * ar] : none;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = sum ? acc + v[u] : fmaxf(acc, v[u]);
    }
    const float x1 = dpp_move_f<kDppQuadSwap1, 0xf>(acc, none);
    acc = sum ? acc + x1 : fmaxf(acc, x1);
    const float x2 = dpp_move_f<kDppQuadSwap2, 0xf>(acc, none);
    acc = sum ? acc + x2 : fmaxf(acc, x2);
    const float x4 = dpp_move_f<kDppHalfMirror, 0xf>(acc, none);
    return sum ? acc + x4 : fmaxf(acc, x4);
}

// The choice j* of a sequence from its best ranking key (0: no eligible
// candidate) and its draft (Sec. 4.3): L = min(K, T-1-j*) when the length is
// valid and 0 <= j* <= T-2, else 0; draft[i] = x[j*+1+i] for i < L, -1 after.
// One wave; `x` is the sequence's token row (global memory or its LDS copy),
// the outputs point at the sequence's own entries.  K = 0: the choice alone.
__device__ __forceinline__ void write_choice_draft(uint64_t best, int64_t T, bool tok_ok,
                                                   const int32_t *x, int K, int32_t *best_pos,
                                                   float *best_score, int32_t *draft,
                                                   int32_t *draft_len) {
    const int lane = lane_id();
    const int32_t bp = best ? (int32_t)(uint32_t)(best & 0xffffffffu) : -1;
    if (lane == 0) {
        *best_pos = bp;
        *best_score = best ? unord_f32((uint32_t)(best >> 32)) : -INFINITY;
    }
    int64_t L = 0;
    if (tok_ok && bp >= 0 && (int64_t)bp <= T - 2) L = min((int64_t)K, T - 1 - bp);
    for (int i = lane; i < K; i += kWave) draft[i] = (i < L) ? x[bp + 1 + i] : -1;
    if (K > 0 && lane == 0) *draft_len = (int32_t)L;
}

// Eq. 2's cosine from the dot product and the two squared norms; the clamp
// is the usual eps = 1e-8 guard (eps^2 on the product of squared norms).
__device__ __forceinline__ float cosine(float dot, float hh, float qq) {
    return dot / sqrtf(fmaxf(hh * qq, 1e-16f));
}

}  // namespace pld
