// Work-item schedule of the persistent attention kernels.
//
// A work item is (sequence s, level c) with 1 <= c <= n_s = ceil(L_s / tile).  The forward and
// the dQ kernel read it as query tile c-1, whose causal span is c key tiles; the dK/dV kernel
// reads it as key tile n_s - c, which c query tiles attend to.  Either way the item's cost is
// proportional to c: the quadratic attention cost of a sequence (paper Sec. 2.1: cost is the sum
// of S_i^2; App. C.2: the quadratic term of T(l,P)) split into a ramp 1..n_s.  The prelude kernel
// writes the items in order of decreasing c.  Persistent workgroups then take items from the
// front of that list through atomic cursors, so the next-longest item always goes to the first
// workgroup that becomes free: longest-processing-time-first list scheduling.
//
// Heads multiply the items.  To keep the workgroups of one XCD (which share an L2) on the same
// K/V heads, the (item, head) space is split into 8 queues, one per XCD; a workgroup drains the
// queue of the XCD it runs on and then steals from the others, so every launch ends with all
// queues empty and no workgroup waits on another.
#pragma once
#include "hyd_device.h"
#include "hyd_rope_regs.h"

namespace hyd {

constexpr int kQueues = 8;
typedef __attribute__((ext_vector_type(4))) int i32x4;

// header (ints): [0] n_items, [1] kSched* flags about cu_seqlens as the prelude saw it, [2] records
// handed out, [3] bytes from here to the header of the list that is handed out in this one's place (0: this one is), [4] bytes from
// here to the records handed out, [5] rows of a tile, [6] heads of a record, the rest zeros; then the cursors of the eight queues, 256 bytes apart: the workgroups of all XCDs claim
// through them with device-scope atomics, which a shared line serialises (one line for all eight:
// forward of 26177 tokens in sequences of 64-1024, 32 heads, d = 64: 227 us, apart 216)
constexpr int kHdrInts = 64, kCursorStride = 64;
constexpr int kHdrCursor = kHdrInts, kHdrTotal = kHdrInts + kQueues * kCursorStride;
constexpr int kHdrFlags = 1, kHdrExec = 2, kHdrOther = 3, kHdrRecords = 4, kHdrTile = 5, kHdrHeads = 6;
constexpr int kSchedTooLong = 1;          // a sequence is longer than max_seqlen: its tiles beyond that bound got no item
constexpr int kSchedBadSeqlens = 2;       // cu_seqlens does not start at 0, does not end at T, or decreases

struct SchedView {            // device pointers into the workspace (all int32)
    int* hdr;                 // kHdrTotal
    int* lev;                 // 3 * (n_lev + 2): level arrays, used instead of LDS when n_lev is large
    int* order;               // n_seq: sequence index by rank (more tiles first, then arrival)
    int* items;               // 4 * max_items : records (s, c, first packed row, length), decreasing c
    int* exec;                // the same records in the order in which they are handed out (see build_schedule); may be `items` itself
    int group_max;            // levels 1 .. group_max at most are grouped by sequence (0 when exec == items)
    float group_share;        // ... and at most (sum of all levels) * group_share
    int n_lev;                // upper bound on tiles per sequence
    int max_items;
    int part_max, part_q, steps_per_level;     // items in parts (see item_parts); part_max = 1: whole
    int other, rec_heads;     // header words kHdrOther, kHdrHeads
    // Two lists of which one is handed out: the one with pick = 1 if wide_pays for the lengths there are, else the one with pick = -1, whose
    // `other` leads to the first (pick = 0: handed out anyway)
    int pick, pick_hkv, pick_wgs;
    long long pick_squares;
};

// dK/dV by tiles of 256 keys: whether sequences with this sum of squared lengths and this longest one are long and even enough (the
// host's rule says why): the sum is at least min_squares, and the longest item at most 1.25 of a workgroup's share.
__host__ __device__ __forceinline__ bool wide_pays(unsigned long long squares, long long longest, long long T, long long min_squares, int hkv, int wgs) {
    return squares >= (unsigned long long)min_squares && 8ull * 256 * (unsigned)wgs * (unsigned long long)longest <= 5ull * (unsigned)hkv * (squares + 256ull * (unsigned long long)T);
}

// An item can be handed out in parts (dK/dV kernel): level c, with c * steps_per_level steps, in
// ceil(steps / part_q) of them, at most part_max.  exec then holds a record per part, which carries its
// index and the number of parts in the level's upper bits.
constexpr int kLevBits = 24, kPartsMax = 8;
__host__ __device__ __forceinline__ int item_parts(int c, int steps_per_level, int part_q, int part_max) {
    if (part_max <= 1) return 1;
    const long long n = ((long long)c * steps_per_level + part_q - 1) / part_q;
    return n < part_max ? (int)n : part_max;
}

struct HeadMap {              // how (item, head) pairs are spread over the queues
    int striped;              // 0: heads partitioned over the queues; 1: items striped
    int heads;                // heads per item (Hq for fwd/dQ, Hkv for dK/dV)
    int hpq;                  // partitioned: heads per queue
    int group;                // partitioned: consecutive work indices share group-size heads
    int grid;                 // workgroups of the launch
};

// In-place inclusive scan of v[0..n) by ONE wave (all 64 lanes call it; n arbitrary): every lane
// sums a contiguous chunk, the chunk sums are scanned across the lanes, each lane rewrites its chunk.
__device__ __forceinline__ void wave_inclusive_scan(int* v, int n, int lane) {
    const int chunk = (n + 63) / 64;
    const int lo = lane * chunk, hi = min(n, lo + chunk);
    __threadfence_block();                 // v was written by other lanes of this wave
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += v[i];
    int run = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(run, d, 64);
        if (lane >= d) run += up;
    }
    run -= sum;
    for (int i = lo; i < hi; ++i) { run += v[i]; v[i] = run; }
    __threadfence_block();                 // and is read by other lanes next
}

constexpr int kPreludeThreads = 1024;
constexpr int kPreludeLdsLev = 4096;      // levels whose arrays fit the kernel's LDS
// bytes of LDS that build_schedule needs for lists of these numbers of levels
inline size_t schedule_lds(int nl0, int nl1, int nl2 = 0, int nl3 = 0) {
    size_t most = 0;
    for (const int nl : {nl0, nl1, nl2, nl3})
        if (nl <= kPreludeLdsLev && sizeof(int) * 3 * (size_t)(nl + 2) > most) most = sizeof(int) * 3 * (size_t)(nl + 2);
    return most;
}

// Builds the item list for tile size `tile` and clears the cursors; called by all `nthreads`
// threads of one workgroup, lds_lev as sized by schedule_lds.  n_lev bounds the tiles per sequence
// (from the caller's max_seqlen).  Order among items of equal cost: by sequence rank (arrival order
// among equals), which is unspecified (it never changes a result: every output element has
// exactly one producer).
//
// The order of execution differs from the list at its cheap end: the items of levels 1 .. C follow
// sequence by sequence (longest sequence first, its highest level first).  In the list the tiles of
// one short sequence lie as far apart as the levels do, and each reads the sequence's K and V (dK/dV:
// Q and dO) from HBM again; next to each other they share them in the L2 of their XCD.  C is what
// keeps a launch balanced: group_max levels (C tiles of a sequence and a head fit the L2 next to
// those of the other workgroups) and a sixteenth of what a workgroup has to do in all, since the last
// items handed out are no longer the cheapest ones.  Measured (forward / dQ / dK/dV in us, list order
// -> this one, 32768 tokens, 32 heads): lengths 64-400 310 / 455 / 475 -> 284 / 412 / 447, 64-1024 366 /
// 522 / 612 -> 353 / 496 / 573, 32 x 1024 435 / 593 / 803 -> 417 / 565 / 717.  With grouped heads (32/8), whose
// workgroups share a stream across the group, it is within 1.5 % either way and left alone; so are
// striped queues, which deal neighbouring items to different XCDs (dealing blocks of eight instead
// gained nothing).
template <bool kPick = false>             // the list may be one of two (`pick` of the view)
__device__ __forceinline__ void build_schedule(const int32_t* __restrict__ cu, int nseq, int T, int tile, const SchedView& sv,
                                               int* lds_lev, int nthreads) {
    const int tid = threadIdx.x;
    const int nl = sv.n_lev;
    int* lev = nl <= kPreludeLdsLev ? lds_lev : sv.lev;
    int* hist = lev;                       // [n]: sequences with exactly n tiles; later the arrival counters
    int* cnt = lev + (nl + 2);             // [r]: sequences with >= nl - r tiles (levels in reversed order)
    int* offs = lev + 2 * (nl + 2);        // [r]: list position after level nl - r
    // behind the levels of cnt and offs: the sum of the squared lengths (8-byte aligned there), the longest one
    unsigned long long* squares = reinterpret_cast<unsigned long long*>(cnt + nl);
    int* longest = offs + nl;
    if (kPick && tid == 0) { *squares = 0; *longest = 0; }
    for (int i = tid; i < nl + 2; i += nthreads) hist[i] = 0;
    for (int i = tid; i < kHdrTotal; i += nthreads) sv.hdr[i] = 0;
    __syncthreads();
    int flags = (tid == 0 && (cu[0] != 0 || cu[nseq] != T)) ? kSchedBadSeqlens : 0;
    float cost = 0.f;                      // sum of all levels
    unsigned long long sq = 0;
    int most = 0;
    for (int s = tid; s < nseq; s += nthreads) {
        const int L = cu[s + 1] - cu[s];
        if (L < 0) flags |= kSchedBadSeqlens;
        if (L > 0 && (L + tile - 1) / tile > nl) flags |= kSchedTooLong;
        const int n = min((L + tile - 1) / tile, nl);
        if (n > 0) atomicAdd(&hist[n], 1);
        cost += 0.5f * (float)n * (float)(n + 1);
        if (kPick) { most = max(most, L); sq += (unsigned long long)max(L, 0) * (unsigned long long)max(L, 0); }
    }
    if (kPick && sq != 0) { atomicAdd(squares, sq); atomicMax(longest, most); }
    if (cost > 0.f) atomicAdd(reinterpret_cast<float*>(hist), cost);        // hist[0] is not a level
    if (flags) atomicOr(&sv.hdr[kHdrFlags], flags);
    __syncthreads();
    int C = min(min(sv.group_max, nl), (int)fminf(*reinterpret_cast<const float*>(hist) * sv.group_share, 1e6f));
    if (tid < 64) {
        // cnt[r] = sum_{n >= nl - r} hist[n]; offs = inclusive scan of cnt
        for (int r = tid; r < nl; r += 64) cnt[r] = hist[nl - r];
        wave_inclusive_scan(cnt, nl, tid);
        for (int r = tid; r < nl; r += 64) offs[r] = cnt[r];
        wave_inclusive_scan(offs, nl, tid);
    }
    __syncthreads();
    const int n_items = nl > 0 ? min(offs[nl - 1], sv.max_items) : 0;
    // more items than any valid cu_seqlens has: positions of the grouped order would lie outside the records
    if (nl > 0 && offs[nl - 1] > sv.max_items) C = 0;
    const bool handed = !kPick || (sv.pick > 0) == wide_pays(*squares, *longest, T, sv.pick_squares, sv.pick_hkv, sv.pick_wgs);
    if (tid == 0) {
        sv.hdr[0] = n_items;
        sv.hdr[kHdrOther] = kPick && handed ? 0 : sv.other;
        sv.hdr[kHdrRecords] = (int)((const char*)sv.exec - (const char*)sv.hdr);
        sv.hdr[kHdrTile] = tile;
        sv.hdr[kHdrHeads] = sv.rec_heads;
    }
    for (int i = tid; i < nl + 2; i += nthreads) hist[i] = 0;
    __syncthreads();
    // rank of a sequence with n tiles = (#sequences with more tiles) + arrival order among equals
    for (int s = tid; s < nseq; s += nthreads) {
        const int L = cu[s + 1] - cu[s];
        const int n = min((L + tile - 1) / tile, nl);
        if (n <= 0) continue;
        const int more = (n < nl) ? cnt[nl - (n + 1)] : 0;
        sv.order[more + atomicAdd(&hist[n], 1)] = s;
    }
    __syncthreads();
    // Level c (reversed index r = nl - c) holds the sequences of rank < cnt[r] at the list
    // positions [offs[r] - cnt[r], offs[r]): one thread per position finds its level by bisection.
    const bool parts = sv.part_max > 1 && nl > 0 && offs[nl - 1] <= sv.max_items;
    if (parts) {
        if (tid < 64) {                        // hist[r]: records handed out up to level nl - r
            for (int r = tid; r < nl; r += 64) hist[r] = cnt[r] * item_parts(nl - r, sv.steps_per_level, sv.part_q, sv.part_max);
            wave_inclusive_scan(hist, nl, tid);
        }
        __syncthreads();
    }
    if (tid == 0) sv.hdr[kHdrExec] = !handed ? 0 : (parts ? hist[nl - 1] : n_items);
    for (int pos = tid; pos < n_items; pos += nthreads) {
        int lo = 0, hi = nl - 1;               // first r with offs[r] > pos
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (offs[mid] > pos) hi = mid; else lo = mid + 1;
        }
        const int rank = pos - (offs[lo] - cnt[lo]), c = nl - lo;
        const int s = sv.order[rank];
        const int a = cu[s], L = cu[s + 1] - a;
        const i32x4 rec = {s, c, a, L};
        *reinterpret_cast<i32x4*>(sv.items + 4 * pos) = rec;
        if (parts) {
            const int n = item_parts(c, sv.steps_per_level, sv.part_q, sv.part_max);
            for (int x = 0; x < n; ++x) {
                const i32x4 part = {s, c | (x << kLevBits) | ((n - 1) << (kLevBits + 3)), a, L};
                *reinterpret_cast<i32x4*>(sv.exec + 4 * (hist[lo] - (cnt[lo] - rank) * n + x)) = part;
            }
        } else if (sv.exec != sv.items) {
            int e = pos;
            if (c <= C) {
                // items of higher levels, then the C lowest levels of the sequences of lower rank
                e = (C < nl ? offs[nl - C - 1] : 0) + min((L + tile - 1) / tile, C) - c;
                for (int x = 1; x <= C; ++x) e += min(rank, cnt[nl - x]);
            }
            *reinterpret_cast<i32x4*>(sv.exec + 4 * e) = rec;
        }
    }
}

// One list per workgroup: blockIdx.x = 0: tile0 -> sv0, blockIdx.x = 1: tile1 -> sv1.  With rope_tab != NULL the
// first workgroup also fills the rotary frequency table of the call (half_d entries, see hyd_rope_regs.h).
__global__ void __launch_bounds__(kPreludeThreads) hyd_schedule_prelude(const int32_t* __restrict__ cu, int nseq, int T,
                                                                       int tile0, SchedView sv0, int tile1, SchedView sv1,
                                                                       double* rope_tab, int half_d, double log2_base) {
    extern __shared__ int lds_lev[];
    if (rope_tab && blockIdx.x == 0) rope_table_fill(rope_tab, half_d, log2_base, threadIdx.x, kPreludeThreads);
    const bool second = blockIdx.x != 0;
    build_schedule(cu, nseq, T, second ? tile1 : tile0, second ? sv1 : sv0, lds_lev, kPreludeThreads);
}

// Query side of an item of the bf16 forward and dQ kernels, 32 rows of a head per wave; rows = 256 >> S.
//   S = 0: 256 rows of one head.
//   S = 1: 128 rows of one head on four of the eight waves, one per SIMD; the others help with the loads.
//     For launches with less than a workgroup's worth of work per CU, which last as long as their longest
//     item: a wave that has its SIMD to itself takes two thirds of the time for a step.
//   S = 2: 64 rows of four query heads of one KV head.  All waves walk the same key tiles, none idles
//     behind the diagonal of another one, and a sequence's last tile pads it to 64 rows instead of 256: a
//     workgroup takes 136 steps of 64 keys instead of 160 for four heads of a 1024-token sequence, 45
//     instead of 84 for 544 tokens.
template <int S>
struct QuerySplit {
    static_assert(S >= 0 && S <= 2, "whole, half, four heads");
    static constexpr int kRows = 256 >> S, kLh = S == 2 ? 2 : 0;      // rows; log2 of the heads
    static constexpr int kTiles = S == 1 ? 2 : 4;                     // 64-row tiles to stage
    __device__ __forceinline__ static int head_of(int wave) { return S == 2 ? wave >> 1 : 0; }
    // first row of a wave; that of an idle wave lies behind every sequence
    __device__ __forceinline__ static int row_of(int wave) { return S == 2 ? 32 * (wave & 1) : (S == 1 && wave >= 4 ? 1 << 30 : 32 * wave); }
    // byte offset of the item's 64-row tile j (tiles by head, then by row) from row 0 of its first head
    __device__ __forceinline__ static uint32_t tile_at(int j, uint32_t row_stride_b, uint32_t row_b) {
        return S == 2 ? (uint32_t)j * row_b : (uint32_t)(64 * j) * row_stride_b;
    }
};

// Number of work indices of queue x.
__device__ __forceinline__ int queue_size(const HeadMap& hm, int n_items, int x) {
    if (hm.striped) return ((n_items - x + kQueues - 1) / kQueues) * hm.heads;
    return n_items * hm.hpq;
}

// Work index w of queue x -> (item index, head).  A partitioned queue walks the item list in
// chunks of chunk_items() items (the list is ordered by decreasing cost, so a chunk holds items of
// similar cost, in a long sequence neighbouring tiles) and, inside a chunk, one head group after
// the other.  The 32 workgroups of an XCD then sit on neighbouring tiles of ONE KV head (times its
// group's query heads) and share the K/V (or Q/dO) tiles they stream in their L2; with the heads
// interleaved per item, a queue with several groups (MHA: every head is its own group) split
// its workgroups over all of them and shared each stream among a fifth as many.  Walking whole
// groups one after the other would share as well but starts the last group's longest items late,
// which unbalances the end of a short launch; chunks keep the order longest-first up to a window
// of one chunk, an eighth of the list at most.  Measured (one process, both orders alternating):
// the MHA configuration 3 gains 4-6 % in every kernel with chunks of 64, the single-buffer
// configuration 2 (67 items in the forward's list) loses 10 % with whole groups or chunks of 64
// and nothing with chunks of 8-16; the GQA configurations, one group per queue, do not change.
__device__ __forceinline__ int chunk_items(int n_items) { return min(64, max(8, n_items >> 3)); }
__device__ __forceinline__ void decode_work(const HeadMap& hm, int n_items, int x, int w, int& item, int& head) {
    if (hm.striped) {
        item = x + kQueues * (w / hm.heads);
        head = w % hm.heads;
    } else {
        const int chunk = chunk_items(n_items);
        const int per_chunk = chunk * hm.hpq;              // work indices of a full chunk
        const int ck = w / per_chunk, r = w - ck * per_chunk;
        const int first = ck * chunk;
        const int per_group = min(chunk, n_items - first) * hm.group;
        const int grp = r / per_group, r2 = r - grp * per_group;
        item = first + r2 / hm.group;
        head = (x + kQueues * grp) * hm.group + r2 % hm.group;
    }
}

// Persistent-workgroup work fetch.  The first item of a workgroup is fixed: workgroup b starts with
// work index b / 8 of queue b % 8 (workgroups are dispatched to the XCDs in turn, so that is the queue
// of its XCD; nothing depends on it).  Later ones are claimed by thread 0 through the queues' atomic
// cursors, which count from the last fixed index on; an index is resolved to (item, head), the
// item's 16-byte record fetched and the result left in LDS for the workgroup.
//
// The chain "cursor atomic -> item record" is two dependent trips to memory, as long as a whole
// short item, so the atomic is taken off the critical path: a kernel calls claim() while it works on
// an item and the result is only looked at in next().  What remains at the end of an item is one
// trip for the record.  A claimed item waits for its claimer, so the claim is made late: with one to
// three items per workgroup, as in small batches, workgroups that claim when an item begins hold
// the next-longest items next to the longest ones.  The fp32 kernels claim inside their tile loop,
// one step before an item's last (fp32 forward, 4096 tokens, 8 heads: 369 us against 499 us).  The
// bf16 kernels, whose tile steps are ten times shorter, claim behind the loop, so that the atomic
// runs under the epilogue (a branch in their loop cost 8-14 %): against a claim at the item's
// start a context-parallel ring takes 6 % less, a 16384-token step 2 %, a 2304-token step with two KV
// heads 14 %.
//
// When its queue is dry a workgroup reads all eight cursors at once and goes on to the next queue that
// still has work, if there is one; if the fixed indices cover all work there is no claim at all.
// Claiming from the eight queues in turn until the last one was dry took 3-12 us at the end of every
// launch: forward of 256 tokens, 32 heads 24.1 us, now 12.3; 2048 tokens, 8 heads 35.6 -> 31.5, dQ 45.3 ->
// 42, dK/dV 40.8 -> 36.5.
// Every workgroup ends when all queues are empty (the cursors only grow).
// Items of up to kShortItem steps have little behind their loop for the atomic to run under, and hold nothing long: they claim before it
// (forward: behind the barrier that ends its loads, which would wait for the atomic).  Forward / backward in us, claim
// behind the loop -> before it: 20000 sequences of three tokens, 8 heads, d = 64 2635 / 6077 -> 2608 / 5938; 65536 of 16 tokens
// 9230 / 21233 -> 9119 / 20843; 2000 of one token, 32/8 heads 1136 / 2105 -> 1115 / 2090.
constexpr int kShortItem = 2;
struct WorkItem { int seq, lev, head, row0, len; };
constexpr int kSlotInts = 16;          // two buffers of 8 ints
struct WorkFetcher {
    int cur;          // slot buffer holding the current item (all threads)
    // the rest is thread 0's
    int queue;        // queue the next claim goes to
    int n_items;
    int claim_w;      // what the atomic of the claim in flight returns (any use of it waits for it: left alone until next())
    bool claimed;     // a claim is in flight
    int nxt_item;     // next item: index (-1: none), head, and its record in flight
    int nxt_head;
    i32x4 nxt_rec;

    // first index of queue x that is claimed through its cursor
    __device__ __forceinline__ static int fixed(const HeadMap& hm, int x) { return (hm.grid - x + kQueues - 1) / kQueues; }

    __device__ __forceinline__ void issue_claim(const HeadMap& hm, int* cursors) {
        claimed = true;
        claim_w = queue_size(hm, n_items, queue) > fixed(hm, queue) ? atomicAdd(&cursors[queue * kCursorStride], 1) : 0x3fffffff;
    }
    // Turns work index w of `queue` into (item, head) of the next item and requests its record.
    __device__ __forceinline__ void resolve(const HeadMap& hm, int* cursors, const int* __restrict__ items, int w) {
        nxt_item = -1;
        nxt_head = 0;
        claimed = false;
        while (w >= queue_size(hm, n_items, queue)) {        // that queue is exhausted
            bool any = false;
#pragma unroll
            for (int x = 0; x < kQueues; ++x) any |= queue_size(hm, n_items, x) > fixed(hm, x);
            if (!any) return;                                // all work was handed out with the launch
            int taken[kQueues];
#pragma unroll
            for (int x = 0; x < kQueues; ++x)
                taken[x] = fixed(hm, x) + __hip_atomic_load(&cursors[x * kCursorStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t open = 0;
#pragma unroll
            for (int x = 0; x < kQueues; ++x) open |= (taken[x] < queue_size(hm, n_items, x) ? 1u : 0u) << x;
            if (!open) return;
            // the next open queue after the present one
            const uint32_t turned = ((open | (open << kQueues)) >> (queue + 1)) & ((1u << kQueues) - 1);
            queue = (queue + __ffs(turned)) & (kQueues - 1);
            w = fixed(hm, queue) + atomicAdd(&cursors[queue * kCursorStride], 1);
        }
        decode_work(hm, n_items, queue, w, nxt_item, nxt_head);
        nxt_rec = *reinterpret_cast<const i32x4*>(items + 4 * nxt_item);
    }
    __device__ __forceinline__ void publish(int* buf) const {
        buf[0] = nxt_item;
        buf[1] = nxt_head;
        if (nxt_item >= 0) { buf[2] = nxt_rec[0]; buf[3] = nxt_rec[1]; buf[4] = nxt_rec[2]; buf[5] = nxt_rec[3]; }
    }
    __device__ __forceinline__ bool read(const int* buf, WorkItem& w) const {
        if (buf[0] < 0) return false;
        w.head = buf[1]; w.seq = buf[2]; w.lev = buf[3]; w.row0 = buf[4]; w.len = buf[5];
        return true;
    }
    // `slot`: kSlotInts ints of LDS.  All threads must call first/next (each contains a barrier).  `wg`: number of the workgroup
    // among the hm.grid that share the queues.
    __device__ __forceinline__ bool first(const HeadMap& hm, const int* __restrict__ hdr, int* cursors,
                                          const int* __restrict__ items, int* slot, WorkItem& w, unsigned wg) {
        cur = 0;
        if (threadIdx.x == 0) {
            queue = wg & (kQueues - 1);
            n_items = hdr[0];
            resolve(hm, cursors, items, wg / kQueues);
            publish(slot);
        }
        __syncthreads();
        return read(slot, w);
    }
    // Claims the item after the current one; all threads may call it, at most once per item.
    __device__ __forceinline__ void claim(const HeadMap& hm, int* cursors) {
        if (threadIdx.x == 0) issue_claim(hm, cursors);
    }
    __device__ __forceinline__ bool next(const HeadMap& hm, int* cursors, const int* __restrict__ items,
                                         int* slot, WorkItem& w) {
        if (threadIdx.x == 0) {
            if (!claimed) issue_claim(hm, cursors);      // an item without steps
            resolve(hm, cursors, items, fixed(hm, queue) + claim_w);
            publish(slot + 8 * (cur ^ 1));
        }
        __syncthreads();        // the next item is visible; everybody is done with the LDS tiles
        cur ^= 1;
        return read(slot + 8 * cur, w);
    }
};

// Launches in which every (item, head) pair has a workgroup of its own need no list: workgroup b takes head b % heads of item
// b / heads, and its waves find the item in cu_seqlens by themselves, one trip to memory instead of a launch and two trips
// (forward of 256 tokens, 32/8 heads: 13.9 us with the list, 10.1; 2048 tokens, 8 heads 28.4 -> 24.3; fp32, 256 tokens, 2
// heads 18.3 -> 13.7).  The lists, for those who read them back (and the fp32 dK/dV kernel), are built
// by workgroups behind those.  For up to kSelfSeqs sequences, four to a lane.
constexpr int kSelfSeqs = 256;
struct SelfSchedule {
    const int32_t* cu;
    int nseq, T, n_work;                  // n_work: workgroups with an item at most
    bool by_level;                        // they do not all run at once (see self_item)
    int heads, tile, n_lev;               // of the items (see build_schedule)
    int n_lists; int tiles[2]; SchedView lists[2];
    double log2_base;                     // rotary embedding: the frequencies are formed in LDS
};
// Item `index` of the sequences' tiles, the same in all lanes of a wave; false if there are fewer.  Where all run at once, sequence by
// sequence.  Else (by_level) the longest first, as from a list: with few heads the later workgroups would hold the longest
// tiles of the last sequences, and those of one level meet on one XCD where the sequences are alike (forward in us, list, sequence
// by sequence, by level: 38400 tokens in sequences of 2000, 1 head 45.3, 71.6, 39.8; 6400 of 2000, 8 heads 44.3, 49.8, 39.1; 4800 of
// 1000, 8 heads 28.8, 31.0, 23.3).
__device__ __forceinline__ bool self_item(const SelfSchedule& ss, int index, WorkItem& w) {
    constexpr int kPer = kSelfSeqs / 64;  // sequences of a lane
    const int lane = threadIdx.x & 63;
    if (ss.by_level) {
        int row[kPer], len[kPer], n[kPer], most = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            row[j] = ss.cu[min(64 * j + lane, ss.nseq)];
            len[j] = ss.cu[min(64 * j + lane + 1, ss.nseq)] - row[j];
            n[j] = min((len[j] + ss.tile - 1) / ss.tile, ss.n_lev);
            most = max(most, n[j]);
        }
        int l = 0, left = index;          // level: first the highest there is, then down to that of the item
        for (int bit = 1 << 16; bit; bit >>= 1)
            if (__ballot(most >= l + bit)) l += bit;
        unsigned long long has[kPer] = {};
        for (; l > 0; --l) {
            int count = 0;
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (64 * j < ss.nseq) { has[j] = __ballot(n[j] >= l); count += __popcll(has[j]); }
            if (left < count) break;
            left -= count;
        }
        if (l == 0) return false;
        w.lev = l;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int count = __popcll(has[j]);
            if (left >= 0 && left < count) {
                const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(has[j] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)has[j], 0u));
                const int src = __ffsll((long long)__ballot(before == left && n[j] >= l)) - 1;
                w.seq = 64 * j + src;
                w.row0 = __builtin_amdgcn_readlane(row[j], src);
                w.len = __builtin_amdgcn_readlane(len[j], src);
            }
            left -= count;                // (below zero once it is found)
        }
        return true;
    }
    int at[kPer + 1], n[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j <= kPer; ++j) at[j] = ss.cu[min(lane * kPer + j, ss.nseq)];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        n[j] = max(min((at[j + 1] - at[j] + ss.tile - 1) / ss.tile, ss.n_lev), 0);
        sum += n[j];
    }
    int run = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(run, d, 64);
        if (lane >= d) run += up;
    }
    int left = index - (run - sum);       // items of this lane's sequences before the wanted one
    const unsigned long long mine = __ballot(left >= 0 && left < sum);
    if (mine == 0) return false;
    int seq = lane * kPer, row0 = at[0], len = at[1] - at[0], tiles = n[0];
#pragma unroll
    for (int j = 0; j + 1 < kPer; ++j)
        if (seq == lane * kPer + j && left >= n[j]) { left -= n[j]; ++seq; row0 = at[j + 1]; len = at[j + 2] - at[j + 1]; tiles = n[j + 1]; }
    const int src = __ffsll((long long)mine) - 1;
    w.seq = __builtin_amdgcn_readlane(seq, src);
    w.lev = __builtin_amdgcn_readlane(tiles - left, src);              // the longest one first
    w.row0 = __builtin_amdgcn_readlane(row0, src);
    w.len = __builtin_amdgcn_readlane(len, src);
    return true;
}
// The workgroup's only item, or its list: false for a workgroup that is done.
__device__ __forceinline__ bool self_first(const SelfSchedule& ss, char* lds, int nthreads, WorkItem& w) {
    if ((int)blockIdx.x >= ss.n_work) {
        const int l = blockIdx.x - ss.n_work;
        build_schedule(ss.cu, ss.nseq, ss.T, ss.tiles[l], ss.lists[l], reinterpret_cast<int*>(lds), nthreads);
        return false;
    }
    w.head = blockIdx.x % ss.heads;
    return self_item(ss, blockIdx.x / ss.heads, w);
}

// Optional per-workgroup trace record: {kernel id << 32 | CU key, start, end, items}.
struct WgTrace {
    unsigned long long* rec;      // nullptr: off
    int capacity;
};
__device__ __forceinline__ void trace_write(const WgTrace& tr, int kernel_id, unsigned long long t0,
                                            unsigned long long n_items_done) {
    if (tr.rec && threadIdx.x == 0) {
        const int per_kernel = tr.capacity / 3;
        const int idx = kernel_id * per_kernel + blockIdx.x;
        if ((int)blockIdx.x < per_kernel) {
            unsigned long long* r = tr.rec + 4 * (size_t)idx;
            r[0] = ((unsigned long long)kernel_id << 32) | (unsigned long long)__smid();
            r[1] = t0;
            r[2] = wall_clock64();
            r[3] = n_items_done;
        }
    }
}

}  // namespace hyd
