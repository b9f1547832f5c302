// bf16 forward kernel: block-diagonal causal flash-style tile loop on MFMA with fp32 accumulation.
//
// Work item = (sequence, query tile, query heads of one KV head), 256 or 128 (row, head) pairs in all (see
// QuerySplit).  A workgroup has 8 waves; a wave owns 32 query rows of one head for the whole item, so
// the online softmax never crosses waves.  K/V tiles of 64 keys travel global -> LDS by direct-to-LDS buffer loads (no staging
// registers, no LDS store instructions) into a ring of three stages shared by the waves: while
// tile t is consumed, tiles t+1 and t+2 are in flight.  One barrier per tile.  The Q rows of an
// item come in the same way and are picked up from LDS as fragments; O leaves through LDS too, so
// that every access to HBM covers whole 256-byte rows.
//
// Orientation.  Scores are computed transposed, S^T[key][q] = K Q^T, so that in the accumulator
// lane map (see mfma32) a lane owns ONE query row (column l%32) and 16 keys per 32-key block:
// the row maximum and row sum are in-lane reductions plus one exchange with the other half of
// the wave, and the softmax statistics are per-lane scalars.  The probabilities then feed
// O^T[d][q] = V^T P^T directly as the B operand (contraction index = key = accumulator row),
// while V^T fragments come out of the row-major V tile with the transposing LDS read.
//
// Reference.  P = exp2(s - m_ref) is exact for ANY per-row reference m_ref as long as nothing
// overflows: bf16 and fp32 keep the relative precision of a probability whatever its size.  So the
// row maximum is taken over the FIRST tile only, and later tiles are not searched for a larger
// score (16 three-way maxima and an exchange per tile and wave, 6 % of the kernel): what a larger
// score does to the row sum l is looked at afterwards.  When l has passed kRefSlack, O and l are
// scaled back by a power of two and m_ref moves up by its exponent (beyond 2^24, where a float no longer
// holds every integer, by what it can, and O and l by as much).  A probability or an O that reaches 2^128
// overflows on the spot; the checks there and, for sums between 2^8 and 2^24, behind the item's last tile find O or l
// non-finite then, and the workgroup repeats the item with care: every tile is searched, and where a
// row's maximum exceeds m_ref by more than 8, O and l are rescaled before the exponentials.  A wave
// goes on with care from its first tile on if the scores of a row there are more than kRefSpread apart: later
// ones are bound to rise then (of 131072 normal scores the largest is 0.45 of the spread of the first 64
// above their maximum, 72 for a spread of 160: this side of that nothing overflows).  Measured, 4 x 4096 tokens, 32
// heads, scores of standard deviation 100 / 40 / 16 nats: 547 / 558 / 584 us; without the look at the spread 1140 /
// 930 / 583; with the maximum of every tile of every item 553 / 561 / 586.  (No probability exceeds a sum below 2^8: O cannot overflow but for the last
// bits of V's range.)  Measured (forward, MI355X): 131072 tokens, 40 heads, d = 128,
// 12.65 -> 12.37 ms; 32768 tokens, 32 heads, d = 64, 1.089 -> 1.033 ms.  Starting the exponentials of key
// block 0 under the score product of block 1, which no longer has to wait for a maximum, is 1.5-4 %
// slower than this order.
//
// Causality.  A wave's 32 rows and the 32-key blocks are aligned, so a block is fully visible,
// fully hidden, or THE diagonal block of the wave (key index in block > row index in block is
// masked).  A wave's diagonal tile is its last, and every tile it computes holds at least one
// visible key for every row, so row maxima are finite.
#pragma once
#include <limits.h>

#include <type_traits>

#include "hyd_sched.h"

namespace hyd {

constexpr int kFwdWaves = 8;
constexpr int kFwdBM = 32 * kFwdWaves, kFwdBN = 64, kFwdThreads = 64 * kFwdWaves;
constexpr int kFwdStages = 3;
constexpr int kFwdTileBytes = kFwdBN * kRowBytes;                 // 16 KB
constexpr int kFwdStageBytes = 2 * kFwdTileBytes;                 // K tile, then V tile
// Q staging: the item's 256 Q rows arrive by direct-to-LDS loads (whole rows per instruction, as
// the K/V tiles do) in four 64-row tiles: two in a region of their own, two in the ring's last
// stage, which no K/V tile needs before the first step.
constexpr int kFwdQxOff = kFwdStages * kFwdStageBytes;
constexpr int kFwdQxBytes = 2 * kFwdTileBytes;
constexpr int kFwdSlotOff = kFwdQxOff + kFwdQxBytes;                  // work slot (64 bytes), then the overflow flag
constexpr int kFwdLds = kFwdSlotOff + 128;
constexpr int kFwdTabOff = kFwdLds, kFwdSelfLds = kFwdTabOff + kHeadDim / 2 * 8;      // rotary frequencies
__device__ __forceinline__ constexpr int fwd_q_stage_off(int j) {
    return j < 2 ? kFwdQxOff + j * kFwdTileBytes : (kFwdStages - 1) * kFwdStageBytes + (j - 2) * kFwdTileBytes;
}
constexpr float kRefSlack = 16777216.f;                           // 2^24, see "Reference"
constexpr float kRefQuiet = 256.f;                                // 2^kRefStep
constexpr float kRefStep = 8.f, kRefSpread = 160.f;               // log2 units

struct FwdParams {
    const uint16_t* q; const uint16_t* k; const uint16_t* v;
    uint16_t* o; float* lse;
    int T, hq, hkv;
    float scale_log2;                 // softmax_scale * log2(e)
    const int* hdr; int* cursors; const int* items;
    HeadMap hm;
    WgTrace tr;
    const int32_t* ranges;            // range variant only: per sequence (q_begin, q_end, kv_begin, kv_end)
    const double* rope_tab;           // NULL, or the rotary frequency table: Q rows are rotated as they are picked up
};

typedef __attribute__((address_space(3))) void lds_void;

// Largest magnitude as a bit pattern; non-finite values have all exponent bits set.
constexpr uint32_t kInfBits = 0x7f800000u;
template <int N>
__device__ __forceinline__ uint32_t largest_bits(const f32x16 (&a)[N]) {
    uint32_t big = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) big = max(big, __float_as_uint(a[i][r]) & 0x7fffffffu);
    return big;
}

// One 64-key tile for the 32 rows of a wave.  There is ONE body for all tiles (separate bodies for
// masked and unmasked tiles make the compiler keep the accumulators twice and copy them at every
// join); only the masking itself sits in a wave-uniform branch.  `diag`: this is the wave's
// diagonal tile (its second 32-key block may be hidden altogether).
// D: head dimension (128 or 64): D/16 contraction steps in the score product, D/32 output blocks.
template <int D>
__device__ __forceinline__ void fwd_tile(int Kt, int Vt, const FragAddr& fa, const bf16x8 (&qf)[D / 16],
                                         f32x16 (&acc_o)[D / 32], float& m_ref, float& l_run, float scale_log2,
                                         int koff, bool diag, int t, int& t_find, bool& overflow) {
    // t_find: the wave's last tile that is searched for row maxima, the first one unless it works with care
    constexpr int NK = D / 16, NDB = D / 32;
    // The instruction order below is pinned with scheduling fences: left alone, the compiler sinks
    // every LDS read next to its use and serialises read -> wait -> MFMA.
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
    {
        // fragment i = (contraction step i/2, key block i%2); reads run kAhead fragments ahead
        constexpr int kAhead = 6;
        bf16x8 kf[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) kf[i] = frag_row(Kt, fa, i & 1, i >> 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * NK; ++i) {
            s[i & 1] = mfma32(kf[i % kAhead], qf[i >> 1], s[i & 1]);
            if (i + kAhead < 2 * NK) kf[i % kAhead] = frag_row(Kt, fa, (i + kAhead) & 1, (i + kAhead) >> 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the first V fragments are requested now, so that their latency hides behind the softmax
    constexpr int kVAhead = 4;
    LdsQueue lq{0};
    ColFrag vf[kVAhead];
#pragma unroll
    for (int i = 0; i < kVAhead; ++i) issue_col(lq, vf[i], Vt, fa, i / NDB, i % NDB);
    __builtin_amdgcn_sched_barrier(0);
    if (diag) {         // hidden keys score -inf (scale_log2 > 0 always, so exp2 turns them into 0)
        // koff = position of the tile's first key slot of this lane minus the lane's query row.
        // It is formed from the tile index, so that these 32 comparisons stay inside this rarely
        // taken branch (as loop invariants they would be hoisted into 64 scalar registers and
        // spilled at every item).
        const int k0 = koff;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * kb + 8 * (r >> 2) + (r & 3) + k0 > 0) s[kb][r] = -INFINITY;
    }
    if (t <= t_find) {
        // row maximum of the raw scores (a negative softmax scale has been folded into the sign of
        // the Q fragments, so the largest raw score is the largest scaled score)
        float mx = s[0][0], lo, hi;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
        both_halves(mx, lo, hi);
        const float cand = fmaxf(lo, hi) * scale_log2;
        if (t == t_find) {
            m_ref = cand;
            float mn = s[0][0];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) mn = fminf(mn, s[kb][r]);
            if (__any(cand - mn * scale_log2 > kRefSpread)) t_find = INT_MAX;
        } else if (__any(cand > m_ref + kRefStep)) {
            const float m_new = fmaxf(m_ref, cand);
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
            m_ref = m_new;
        }
    }
    // P V: the exponentials of key step b+1 (8 scores) issue under the NDB MFMAs of step b (two
    // scores per MFMA for D = 128, four for D = 64); V fragments are read kVAhead MFMAs ahead.
    float lsum = 0.f;
    auto exp_pair = [&](int j) -> uint32_t {           // scores 2j, 2j+1 of the 32 a lane holds
        const int kb = j >> 3, r = (2 * j) & 15;
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][r], scale_log2, -m_ref));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][r + 1], scale_log2, -m_ref));
        const uint32_t pair = pack_bf16(p0, p1);
        // row sum of the ROUNDED probabilities (what the P V product actually uses)
        bf16x2 pr;
        __builtin_memcpy(&pr, &pair, 4);
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, lsum, false);
        return pair;
    };
    u32x4 pcur, pnxt;
#pragma unroll
    for (int e = 0; e < 4; ++e) pcur[e] = exp_pair(e);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4 * NDB; ++i) {                 // i = NDB*b + db
        const int b = i / NDB, db = i % NDB;
        acc_o[db] = mfma32(lds_wait(lq, vf[i % kVAhead]), as_bf16x8(pcur), acc_o[db]);
        if (i + kVAhead < 4 * NDB) issue_col(lq, vf[i % kVAhead], Vt, fa, (i + kVAhead) / NDB, (i + kVAhead) % NDB);
        if (b < 3) {
#pragma unroll
            for (int e = 0; e < 4 / NDB; ++e) pnxt[(4 / NDB) * db + e] = exp_pair(4 * (b + 1) + (4 / NDB) * db + e);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (db == NDB - 1) pcur = pnxt;
    }
    l_run += lsum;
    if (__builtin_expect(__any(l_run > kRefSlack), 0)) {
        float lo, hi;
        both_halves(l_run, lo, hi);                    // O is shared by the halves of a row, so its scale is too
        const uint32_t e = __float_as_uint(fmaxf(lo, hi)) >> 23;       // l > 0: biased exponent
        const uint32_t big = max(e << 23, largest_bits(acc_o));
        // O and l are scaled by what the reference moves: by 2^-k, unless m_ref is so large that it holds no such
        // sum.  2^-126 is the smallest power of two with an exponent of its own; more is left to the repeat.
        const int k = e > 127u ? min((int)e - 127, 126) : 0;
        const float m_new = m_ref + (float)k, moved = m_new - m_ref;
        const bool ok = big < kInfBits && moved <= 126.f;
        const float alpha = ok ? __builtin_amdgcn_exp2f(-moved) : 1.f;
        if (!ok) overflow = true;
        l_run *= alpha;
        m_ref = ok ? m_new : m_ref;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc_o[db][r] *= alpha;
    }
}

__device__ __forceinline__ double self_log2_base(const SelfSchedule& ss) { return ss.log2_base; }

// R: range variant.  Each sequence has a query range [q_begin, q_end) and a key range
// [kv_begin, kv_end) in local positions, the begins multiples of the query tile: query tiles
// outside the query range are skipped, the tile loop starts at the key range's first tile and
// stops at its end, and a row that sees no key of the range gets O = 0 and LSE = -inf (the
// neutral element of the log-sum-exp merge of partial results).
// With a SelfSchedule as second argument: one item per workgroup, found by itself.  (Both are this kernel and not a function that two
// kernels call: inlined, the compiler hoists the fetcher's divisions and orders the code in front of the tile loop otherwise, 0.3-0.6
// us of every forward that takes a list; 65536 tokens, 32 heads 2870.7 -> 2864.9 us, 9000 tokens, 8 heads 36.0 -> 35.8.)
template <bool R, int D = kHeadDim, int S = 0, typename... SS>
__global__ void __launch_bounds__(kFwdThreads, 1) hyd_fwd_bf16_kernel(FwdParams p, SS... ss) {
    constexpr bool kSelf = sizeof...(SS) != 0;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    using QS = QuerySplit<S>;
    static_assert(D == 128 || D == 64, "head dimension");
    constexpr int kRowB = D * 2;                                      // bytes of a row in global memory
    static_assert(kFwdBM == 256 && kFwdStages == 3, "the Q staging assumes a 256-row tile and a free third stage");
    int* slot = reinterpret_cast<int*>(smem + kFwdSlotOff);
    volatile int* redo = slot + 16;                                            // a wave of the workgroup has overflowed
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const int64_t q_stride = (int64_t)p.hq * D, kv_stride = (int64_t)p.hkv * D;
    const uint32_t kv_stride_b = (uint32_t)kv_stride * 2, q_stride_b = (uint32_t)q_stride * 2;
    const unsigned long long t_start = p.tr.rec ? wall_clock64() : 0ull;
    unsigned long long n_done = 0;

    FragAddr fa;
    fa.init(lane, smem);
    // direct-to-LDS tile load: instruction j of wave w fills tile rows 4*(j*NW + w) .. +3 (1 KB,
    // lane i -> row i/16, chunk position i%16), so lane i fetches the chunk that swz() puts there
    const int dma_row = 4 * wave + (lane >> 4);
    const uint32_t dma_voff = dma_lane_voff<D>(dma_row, lane, kv_stride_b);
    const uint32_t dma_voff_q = dma_lane_voff<D>(dma_row, lane, q_stride_b);
    const uint32_t tile_bytes = kFwdBN * kv_stride_b;                 // one K/V tile in global memory
    // this wave's 32 Q rows inside the staging area, and its private 8 KB of the (free) ring for O
    const int q_stage = ((wave >> 1) < 2 ? kFwdQxOff + (wave >> 1) * kFwdTileBytes
                                         : (kFwdStages - 1) * kFwdStageBytes + ((wave >> 1) - 2) * kFwdTileBytes) +
                        (wave & 1) * 32 * kRowBytes;
    const uint32_t o_stage = (uint32_t)(uintptr_t)(lds_char*)smem + (uint32_t)(wave * 32 * kRowBytes);   // absolute LDS address
    // scale * s = |scale| * (-s): a negative scale flips the sign bits of the Q fragments instead
    // (and a zero scale becomes a denormal-free epsilon, so that -inf * scale stays -inf)
    const float scale_log2 = fmaxf(fabsf(p.scale_log2), 1e-30f);
    const uint32_t sign_flip = p.scale_log2 < 0.f ? 0x80008000u : 0u;

    WorkFetcher wf;
    WorkItem wi;
    bool have;
    if constexpr (kSelf) have = self_first(ss..., smem, kFwdThreads, wi);
    else have = wf.first(p.hm, p.hdr, p.cursors, p.items, slot, wi, blockIdx.x);
    while (have) {
        ++n_done;
        const int lev = wi.lev, head0 = wi.head << QS::kLh, row0 = wi.row0, L = wi.len;
        const int q0 = (lev - 1) * QS::kRows;
        int Lq = L, kb = 0, kcap = L;                     // query rows [.., Lq), keys [kb, kcap)
        if (R) {
            const i32x4 rg = *reinterpret_cast<const i32x4*>(p.ranges + 4 * wi.seq);
            Lq = min(L, rg[1]); kb = max(rg[2], 0); kcap = min(L, rg[3]);
            if (q0 < rg[0] || q0 >= Lq) {                 // the whole query tile is outside the range
                have = wf.next(p.hm, p.cursors, p.items, slot, wi);
                continue;
            }
        }
        const int kv_end = min(kcap, q0 + QS::kRows);
        const int n_kt = (kv_end + kFwdBN - 1) / kFwdBN;
        const int t_lo = R ? kb / kFwdBN : 0;             // first key tile
        const int g = head0 / G;
        const int head = head0 + QS::head_of(wave);      // this wave's query head
        const int wrow0 = q0 + QS::row_of(wave);         // and its first query row
        const int qrow = wrow0 + l32;
        const bool qvalid = qrow < Lq;
        const bool active = wrow0 < Lq;                   // else the wave only helps with the loads
        if (R && kv_end <= kb) {                          // no key of the range is visible to this tile
            if (qvalid) {
                uint16_t* op = p.o + (int64_t)(row0 + qrow) * q_stride + (int64_t)head * D + 4 * half;
                const u32x2 z = {0u, 0u};
#pragma unroll
                for (int i = 0; i < D / 8; ++i) *reinterpret_cast<u32x2*>(op + 8 * i) = z;
                if (half == 0) p.lse[(int64_t)head * p.T + row0 + qrow] = -INFINITY;
            }
            have = wf.next(p.hm, p.cursors, p.items, slot, wi);
            continue;
        }
        int td = wrow0 / kFwdBN;                          // this wave's diagonal (= last) tile
        // An item that the waves found by themselves is the workgroup's to the compiler too, and it would make the branches on the
        // diagonal scalar and keep the accumulators twice, copied in every tile (see fwd_tile): one sequence of 65280 tokens, 1 head
        // 1428 us from a list, 1559 so, 1438 now; 2040 tokens, 32/8 heads 58.2 and 57.1, now 53.5.
        if constexpr (kSelf) asm volatile("" : "+v"(td));
        const int koff0 = 4 * half - qrow;                // first key slot of the lane minus its query row, tile 0
        // K/V rows [0, kv_end) of this sequence and KV head; reads past them return zero
        const uint32_t kv_bytes = (uint32_t)(kv_end - 1) * kv_stride_b + kRowB;
        const __amdgpu_buffer_rsrc_t rk = make_rsrc(p.k + (int64_t)row0 * kv_stride + (int64_t)g * D, kv_bytes);
        const __amdgpu_buffer_rsrc_t rv = make_rsrc(p.v + (int64_t)row0 * kv_stride + (int64_t)g * D, kv_bytes);
        auto dma_tile = [&](int t, int stage) {
            char* dst = smem + stage * kFwdStageBytes + 4 * wave * kRowBytes;
#pragma unroll
            for (int j = 0; j < 16 / kFwdWaves; ++j) {
                const uint32_t soff = (uint32_t)t * tile_bytes + (uint32_t)(j * kFwdWaves * 4) * kv_stride_b;
                char* d = dst + j * kFwdWaves * 4 * kRowBytes;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void*)d, 16, dma_voff, soff, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(d + kFwdTileBytes), 16, dma_voff, soff, 0, 0);
            }
        };
        dma_tile(t_lo, 0);
        if (t_lo + 1 < n_kt) dma_tile(t_lo + 1, 1);

        {   // the item's Q rows; rows past the query range read as zeros (the last row ends with its last head)
            const uint32_t q_bytes = (uint32_t)(min(Lq - q0, QS::kRows) - 1) * q_stride_b + (kRowB << QS::kLh);
            dma_rows<kFwdWaves>(make_rsrc(p.q + (int64_t)(row0 + q0) * q_stride + (int64_t)head0 * D, q_bytes), smem,
                                [](int j) { return fwd_q_stage_off(j); }, QS::kTiles, q_stride_b,
                                [&](int j) { return QS::tile_at(j, q_stride_b, kRowB); }, wave, dma_voff_q);
        }
        if (tid == 0) *redo = 0;
        if constexpr (kSelf) {
            if (p.rope_tab) rope_table_fill(reinterpret_cast<double*>(smem + kFwdTabOff), D / 2, self_log2_base(ss...), tid, kFwdThreads);
        }
        __syncthreads();                                  // the first tiles and the Q rows have landed
        bf16x8 qf[D / 16];
        {
            u32x4 qv[D / 16];
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) qv[ks] = *(lds_u32x4*)(uintptr_t)(fa.row[ks] + (uint32_t)q_stage);
            __builtin_amdgcn_s_waitcnt(0xc07f);           // lgkmcnt(0)
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) {
                asm volatile("" : "+v"(qv[ks]));          // the reads stay on this side of the barrier
            }
            if (p.rope_tab) rope_row_frags<D, false>(qv, kSelf ? reinterpret_cast<const double*>(smem + kFwdTabOff) : p.rope_tab, qrow, half);      // position = local row: reset per sequence
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) qf[ks] = as_bf16x8(qv[ks] ^ sign_flip);
        }
        __builtin_amdgcn_s_barrier();                     // the staged Q may be overwritten (tile t_lo+2 goes there)
        const bool short_item = n_kt - t_lo <= kShortItem;
        if (!kSelf && short_item) wf.claim(p.hm, p.cursors);

        f32x16 acc_o[D / 32];
        float m_ref, l_run;
        bool overflow = false;
        int t_find = t_lo;       // last tile that is searched for row maxima
        while (true) {
            m_ref = -INFINITY;
            l_run = 0.f;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[db][r] = 0.f;
            // one tile on ring stage ST (compile-time, so that fragment reads are base+immediate)
            auto step = [&](auto stage_tag, int t) {
                constexpr int ST = decltype(stage_tag)::value;
                constexpr int Kt = ST * kFwdStageBytes, Vt = Kt + kFwdTileBytes;      // LDS offsets of the tiles
                // the loads run two tiles ahead: tile t+1 was requested one step ago and precedes this
                // step's loads in the (in-order) vmcnt queue
                constexpr int ST2 = (ST + 2) % kFwdStages;
                constexpr int kDmaPerTile = 2 * (16 / kFwdWaves);
                const bool more2 = t + 2 < n_kt;
                if (more2) dma_tile(t + 2, ST2);
                if (active && t <= td)
                    fwd_tile<D>(Kt, Vt, fa, qf, acc_o, m_ref, l_run, scale_log2, t * kFwdBN + koff0, t == td,
                                t, t_find, overflow);
                if (more2) __builtin_amdgcn_s_waitcnt(0x0070 | (kDmaPerTile & 15));     // vmcnt(kDmaPerTile), lgkmcnt(0)
                else __builtin_amdgcn_s_waitcnt(0x0070);                                // vmcnt(0), lgkmcnt(0)
                __builtin_amdgcn_s_barrier();
            };
            for (int t = t_lo; t < n_kt; t += 3) {
                step(std::integral_constant<int, 0>{}, t);
                if (t + 1 < n_kt) step(std::integral_constant<int, 1>{}, t + 1);
                if (t + 2 < n_kt) step(std::integral_constant<int, 2>{}, t + 2);
            }
            // (behind the loop, with a barrier of its own: in the last step it cost the long items 1 %)
            if (__any(l_run > kRefQuiet)) overflow |= largest_bits(acc_o) >= kInfBits;
            if (t_find == t_lo && __any(overflow)) *redo = 1;
            __syncthreads();
            if (__builtin_expect(*redo == 0, 1)) break;
            t_find = INT_MAX;
            __syncthreads();
            if (tid == 0) *redo = 0;
            dma_tile(t_lo, 0);
            if (t_lo + 1 < n_kt) dma_tile(t_lo + 1, 1);
            __syncthreads();
        }
        if (!kSelf && !short_item) wf.claim(p.hm, p.cursors);
        // epilogue: normalise, write O (bf16) and LSE (natural log)
        float l_lo, l_hi;
        both_halves(l_run, l_lo, l_hi);
        const float l_tot = l_lo + l_hi;
        // range variant: a row below the key range has l = 0, m = -inf: O = 0, LSE = -inf
        const float inv = (R && !(l_tot > 0.f)) ? 0.f : 1.f / l_tot;
        if (active) {
            // O leaves through this wave's 8 KB of the ring (free now): whole rows per store
            store_rows_via_lds<D>(p.o + (int64_t)(row0 + wrow0) * q_stride + (int64_t)head * D, q_stride, Lq - wrow0,
                               acc_o, inv, o_stage, lane);
            if (qvalid && half == 0)
                p.lse[(int64_t)head * p.T + row0 + qrow] =
                    (m_ref + __builtin_amdgcn_logf(l_tot)) * 0.69314718055994530942f;
        }
        if constexpr (kSelf) have = false;
        else have = wf.next(p.hm, p.cursors, p.items, slot, wi);
    }
    trace_write(p.tr, 0, t_start, n_done);
}

}  // namespace hyd
