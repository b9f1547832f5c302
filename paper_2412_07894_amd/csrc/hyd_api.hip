// Host side of the C ABI declared in include/hyd_attn.h: argument validation (before any HIP
// call), workspace layout, launch configuration and the benchmark hooks.
#include "../../include/hyd_attn.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <mutex>
#include <vector>

#include "hyd_bwd_bf16.h"
#include "hyd_bwd_wide.h"
#include "hyd_fp32.h"
#include "hyd_fwd_bf16.h"
#include "hyd_fwd_coop.h"
#include "hyd_merge.h"
#include "hyd_rope.h"

namespace {

using namespace hyd;

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Workspace: one schedule, two for the backward (dK/dV, dQ), then the backward's row statistics ([Hq][T] floats; the fp32 path uses the
// first one only) and, for bf16, the fp16 copies of Q, dO and K that its tile loops stream.
constexpr int kBwdStatVecs = 4;
struct SchedLayout { size_t hdr, lev, order, items, exec; int n_lev, max_items; };
struct WsLayout {
    SchedLayout sched[2];
    SchedLayout split;      // query side by QuerySplit tiles, where an item is not a whole tile (split > 0)
    SchedLayout wide;       // bf16 backward: dK/dV by tiles of kKwBN keys
    int n_sched;
    int part_max;           // dK/dV items in parts: their number at most
    // used: what the call uses; need: what it demands; the parts' sums take what lies behind, up to total (see part_bytes)
    size_t stat[kBwdStatVecs], q16, do16, k16, absmax, rope_tab, used, need, total;
};
constexpr int kRopeTabEntries = 64;       // head_dim / 2 at most

// levels of a sequence of `len` rows, in whole multiples of 2^split tiles: a list of split tiles covers
// the same rows as the list of whole ones for every bound on the sequence length
int levels(int len, int tile, int split) {
    const int whole = tile << split, n = (len + whole - 1) / whole;
    return (n < 1 ? 1 : n) << split;
}

// `compact`: the records are handed out in list order, without a second copy of them
size_t sched_layout(SchedLayout& v, size_t at, int T, int nseq, int tile, int split, bool compact, int part_max = 1) {
    v.n_lev = levels(T, tile, split);
    v.max_items = T / tile + nseq + 1;
    v.hdr = at;   at += align_up(sizeof(int) * kHdrTotal);
    v.lev = at;   at += align_up(sizeof(int) * 3 * (size_t)(v.n_lev + 2));
    v.order = at; at += align_up(sizeof(int) * (size_t)(nseq > 0 ? nseq : 1));
    v.items = at; at += align_up(sizeof(int) * 4 * (size_t)v.max_items);
    v.exec = v.items;
    if (!compact) { v.exec = at; at += align_up(sizeof(int) * 4 * (size_t)v.max_items * (size_t)part_max); }
    return at;
}

// Batches of up to so many (token, head) pairs run dK/dV beside dQ in one launch: each of the two leaves most of the chip
// idle and lasts as long as its longest item.  dK/dV converts dO itself then, which costs it a fifth where the chip is
// full.  Backward, one launch after the other -> beside each other (log-normal lengths, d = 128): 8 heads, 1500 tokens 70 -> 51
// us, 3000 tokens 103 -> 80, 6000 184 -> 164 (8/1 heads 187 -> 191, one sequence 318 -> 383); 32 heads, 700 tokens 56 -> 48, 1500
// 93 -> 86 (32/8 heads 94 -> 94), 3000 200 -> 208.
constexpr long long kBothRows = 40960;
// With three or more query heads per KV head the fifth weighs more, since such items go in parts of many steps: one sequence that nearly
// fills the limit loses.  So `heads` times a workgroup's share of the steps stays within 300, which is 35000 pairs for one
// sequence, and no limit where several hold them (one after the other -> beside each other: one sequence of 13600 tokens, 3/1 heads
// 565 -> 608, 6800, 6/2 312 -> 329, 6/1 301 -> 330, 5800, 7/1 270 -> 277, 1280, 32/1 175 -> 183, 600, 64/1 164 -> 179; 10000, 3/1 398 -> 364,
// 5000, 6/2 223 -> 202, 4000, 8/1 197 -> 159; with two, 20480, 2/1 896 -> 838; with one, 40960, 1 head 1881 -> 1654).
constexpr double kBothHeadShares = 300;

// Parts of dK/dV items.  An item may be taken in as many parts as the sums of all rows fit behind the rest of the
// workspace and into kPartBytes (splitting pays where few items keep few compute units busy, which needs a small
// batch or few KV heads).  A call with a smaller workspace takes fewer parts or none: a workspace made for more tokens does for
// fewer, whatever a batch could use.  What a batch can use at most, whatever its max_seqlen, is a maximum over the number
// of key tiles of its longest sequence, so that the size asked for never falls as tokens are added.
constexpr size_t kPartBytes = 256u << 20;
constexpr int kPartSteps = 16;                             // see set_parts
constexpr int kBothPartSteps = 4, kBothPartGain = 8;       // see both_parts
constexpr size_t kBothPartBytes = 64u << 20;
size_t part_bytes(int T, int hkv, int head_dim) { return 2 * sizeof(float) * (size_t)T * (size_t)hkv * (size_t)head_dim; }
int part_limit(size_t bytes, int T, int hkv, int head_dim) {
    const size_t one = part_bytes(T, hkv, head_dim);
    int n = hkv <= 65535 ? kPartsMax : 1;                  // KV heads are a grid dimension of the summing kernel
    while (n > 1 && (size_t)n * one > kPartBytes) n >>= 1;
    return (size_t)n * one <= bytes ? n : (int)(bytes / one < 1 ? 1 : bytes / one);
}
double share_of_work(double tile, double steps_per_level, int T, int nseq, int max_seqlen, int heads, int wgs) {
    const double nm = max_seqlen / tile, m = nseq > 1 ? nseq - 1 : 1, nr = (T - max_seqlen) / m / tile;
    return heads * steps_per_level * (nm * (nm + 1) + m * nr * (nr + 1)) / 2 / wgs;
}
bool both_ok(int T, int nseq, int max_seqlen, int hq, int hkv, int cus) {
    return (long long)T * hq <= kBothRows &&
           (hq < 3 * hkv || hq * share_of_work(kKvBN, kKvBN / kKvBM * (hq / hkv), T, nseq, max_seqlen, hkv, cus) <= kBothHeadShares);
}
// steps of a part, 0: items stay whole (see set_parts)
double steps_of_part(double longest, double share, int limit) {
    if (limit <= 1 || longest < 1.6 * share || longest < 2 * kPartSteps) return 0;
    const double q = share / 2 > kPartSteps ? share / 2 : kPartSteps;
    return q < longest / limit ? longest / limit : q;
}
size_t useful_part_bytes(int T, int hq, int hkv, int head_dim) {
    if (hkv > 65535) return 0;
    const int steps = kKvBN / kKvBM * (hq / hkv), levels = (T + kKvBN - 1) / kKvBN;
    int most = 1;
    for (int n = 1; n <= levels && most < kPartsMax; ++n) {        // the longest sequence has n tiles, and nothing lies beside it
        const double share = share_of_work(kKvBN, steps, (n - 1) * kKvBN + 1, 1, (n - 1) * kKvBN + 1, hkv, 256);
        const double q = steps_of_part((double)n * steps, share, kPartsMax);
        if (q > 0 && most < (int)ceil(n * steps / q)) most = (int)ceil(n * steps / q);
        if ((double)n * steps < 1.6 * share) break;                 // and so on: a share grows with n squared
    }
    size_t bytes = most == 1 ? 0 : (size_t)most * part_bytes(T, hkv, head_dim);
    const int both = T < kBothRows / hq ? T : (int)(kBothRows / hq);        // tokens of the largest batch that both_parts takes
    if (steps * ((both + kKvBN - 1) / kKvBN) >= kBothPartSteps + kBothPartGain) {
        const int parts = hq / hkv < 4 ? 2 * (hq / hkv) + 1 : kPartsMax;     // (a part has a step per key tile of the item at least)
        const size_t some = (size_t)parts * part_bytes(both, hkv, head_dim), room = some < kBothPartBytes ? some : kBothPartBytes;
        if (bytes < room) bytes = room;
    }
    return bytes < kPartBytes ? bytes : kPartBytes;
}

// split: finest form of the query side's items (the last list).  The list of whole tiles has its order of
// execution only where that differs from it (make_view).
WsLayout ws_layout(int T, int nseq, int tile0, int tile1, int split, int hq, int hkv, int head_dim, hyd_dtype dt, bool bwd, bool compact = false, size_t bytes = 0) {
    WsLayout w;
    const size_t useful = bwd && dt == HYD_BF16 ? useful_part_bytes(T, hq, hkv, head_dim) : 0;
    size_t at = sched_layout(w.sched[0], 0, T, nseq, tile0, 0, compact || (!bwd && hq >= 4 * hkv), useful ? kPartsMax : 1);
    w.n_sched = bwd ? 2 : 1;
    if (bwd) at = sched_layout(w.sched[1], at, T, nseq, tile1, 0, hq >= 4 * hkv);
    else w.sched[1] = w.sched[0];
    if (split > 0) at = sched_layout(w.split, at, T, nseq, (bwd ? tile1 : tile0) >> split, split, true);
    else w.split = w.sched[1];
    if (bwd && dt == HYD_BF16) at = sched_layout(w.wide, at, T, nseq, kKwBN, 0, hq >= 4 * hkv);
    else w.wide = w.sched[0];
    const int n_stat = !bwd ? 0 : (dt == HYD_BF16 ? kBwdStatVecs : 1);
    for (int i = 0; i < kBwdStatVecs; ++i) {
        w.stat[i] = at;
        if (i < n_stat) at += align_up(sizeof(float) * (size_t)T * (size_t)hq);
    }
    const bool copies = bwd && dt == HYD_BF16;
    w.q16 = at;  if (copies) at += align_up(2 * (size_t)T * (size_t)hq * (size_t)head_dim);
    w.do16 = at; if (copies) at += align_up(2 * (size_t)T * (size_t)hq * (size_t)head_dim);
    w.k16 = at;  if (copies) at += align_up(2 * (size_t)T * (size_t)hkv * (size_t)head_dim);
    w.absmax = at; if (copies) at += align_up(sizeof(uint32_t) * kPrepMaxWg);
    w.rope_tab = at; at += align_up(sizeof(double) * kRopeTabEntries);       // rotary frequency table (the *_rope calls)
    w.used = w.need = at;
    w.total = at + align_up(useful);
    w.part_max = useful && bytes > at ? part_limit(bytes - at, T, hkv, head_dim) : 1;
    return w;
}

// rows per work item of the forward and dQ kernels (over all of its heads) and of the dK/dV kernel
static_assert(kFwdBM == 256 && kDqBM == 256, "QuerySplit");
int tile_q(hyd_dtype dt) { return dt == HYD_BF16 ? 256 : kF32BM; }
int tile_kv(hyd_dtype dt) { return dt == HYD_BF16 ? kKvBN : kF32KvBN; }
// Form of the query side's items (QuerySplit) in a call without ranges.
//
// Half tiles where a launch lasts as long as its longest item: that item's steps are 2.5 times a
// workgroup's share of all steps or more, the work bounded from below as in set_parts.  (Half / whole,
// forward and dQ, log-normal lengths unless noted: 8 heads, 2048 tokens, 7 shares 0.85 / 0.82, 4096 tokens, 4.4
// shares 0.72 / 0.75, 8192 tokens, 2.9 shares 0.69 / 0.69; 10 heads, one sequence of 4096, 3.0 shares 0.70 /
// 0.71; 32 heads, 1536 tokens, 2.5 shares 0.83 / 0.82; 8 heads, 8192 tokens of 64-1024, 2.4 shares 1.08 / 1.02; 32
// heads, 2048 tokens, 1.75 shares 1.05 / 1.04, 4096 tokens, 1.1 shares 1.20 / 1.15.)
//
// Four heads per item where the query heads of a KV head come in fours and there
// are items for two rounds of workgroups.  With fewer, a launch lasts as long as its longest items,
// and those are shorter with 256-row tiles, whose waves drop out one by one on the diagonal (32/8 heads,
// log-normal lengths, forward / dQ in us, whole -> four heads: 2048 tokens 37.1 / 51.1 -> 40.2 / 54.1; 4096
// tokens 99.5 / 137.6 -> 99.0 / 136.2; 6144 143.8 / 202 -> 140.8 / 197.5; 32768 tokens of 64-1024 336.5 /
// 478 -> 319 / 452; 64/8 heads, 16384 tokens 654 / 885 -> 612 / 852; 16/2 heads, 32768 tokens 449 / 594 ->
// 421 / 569).  The range variants, whose rows are a part of the tokens, keep whole tiles (a
// context-parallel ring of four, 16384 tokens: 2980 us, four heads 3018).
//
// `compact`: whole tiles, which need the fewest records.
constexpr long long kFourHeadPairs = 2 * 256 * 256;        // (token, head) pairs of two items for each of 256 CUs
int query_split(hyd_dtype dt, int T, int nseq, int max_seqlen, int hq, int hkv, bool compact) {
    if (dt != HYD_BF16 || compact) return 0;
    const double steps = 256 / kFwdBN;                     // per level of a whole tile
    if (max_seqlen / 256.0 * steps >= 2.5 * share_of_work(256, steps, T, nseq, max_seqlen, hq, 256)) return 1;
    return (hq / hkv) % 4 == 0 && (long long)T * hq >= kFourHeadPairs ? 2 : 0;
}
// the finest tile that a call of these sizes may choose, for the workspace
int finest_split(hyd_dtype dt, int hq, int hkv, bool compact) {
    return dt != HYD_BF16 || compact ? 0 : ((hq / hkv) % 4 == 0 ? 2 : 1);
}
// dK/dV by tiles of 256 keys (hyd_bwd_wide.h) instead of 128.  The host knows T, the number of sequences and a bound on
// their length: with one sequence of that length and the others alike, `mean` is the length of a token's sequence on average
// and `share` a workgroup's share of the work.
//   Length: a step of the wide form is a fifth cheaper, an item's beginning and end are not hidden.  Equal sequences, 49152 tokens,
// backward narrow -> wide in us, 32 heads, d = 128: 512 tokens 1585 -> 1590, 900 2099 -> 2127, 1300 2673 -> 2619, 2048 3530 -> 3362;
// 32/8 heads, whose items are four times as long: 300 1115 -> 1171, 400 1277 -> 1286, 640 1472 -> 1425, 1024 1981 -> 1852; 32 heads,
// d = 64: 300 1072 -> 1108, 400 1088 -> 1056, 1024 1380 -> 1287.
//   Number: its longest item takes twice as long.  Backward, log-normal lengths unless noted, longest / share: 50000 tokens, 8 heads,
// 1.04: 1014 -> 981; 24000 tokens of Pareto lengths, 8 heads, 1.29: 1014 -> 1024; one sequence of 12000, 32/8 heads, 1.34: 3705 ->
// 3728; 12000 tokens of Pareto lengths, 32/8 heads, 1.63: 2520 -> 2729; 12000 tokens, 32/8 heads, 2.1: 897 -> 1047.
//   Rounds: with few items of about one length for each workgroup the last round is half empty, or an item late, and lasts twice as long as in
// the narrow form.  Backward, equal lengths: 12000 tokens (1.5 items for each workgroup): 700 long, 32/8 heads, d = 128 405 -> 432, 64/8 740 -> 771,
// 1000, 32/8 477 -> 484; d = 64: 500, 32/8 219 -> 236, 64/8 398 -> 436, 16/8 120 -> 129, 1000, 32/8 306 -> 297; 12000 (1.8), 10 heads, d = 128: 2500
// 322 -> 331; 16384 (2), 32/8: 640 509 -> 536, 1000 670 -> 692; 24000 (3), 32/8: 700 776 -> 796, 1000 961 -> 938; 8 heads, d = 64 700 170 -> 173;
// 50000 (6), 8 heads, d = 64: 500 302 -> 305, 700 335 -> 329.
//   Heads: with three or more of them for a queue, a workgroup's items come by heads in windows of eight records (decode_work), and the long ones of
// the later heads begin late.  With less than 2.4 (d = 128: 3.1) items for each workgroup that outweighs the gain (dK/dV, narrow -> wide, items
// for each): 32 heads, 3713 tokens, d = 128 (1.8) 230 -> 251, [1834, 1419], d = 64 (1.6) 74 -> 83; 48 heads, d = 64, 2373 (1.7) 105 -> 125, 2743 (2.0)
// 128 -> 143, 3209 (2.4) 170 -> 174, 3051, 64 heads (3.0) 203 -> 194; d = 128, 40 heads [2804, 1029] (2.3) 190 -> 210, 48, 4122 (3.0) 398 -> 406, 40, 5417
// (3.3) 556 -> 534; with fewer heads: 16, [3812, 3676] (1.9) 228 -> 228, 8279 (2.1) 518 -> 499.
// The range variants, whose visits are a part of these items, keep the narrow form, and so do items in parts.
//   A bound: max_seqlen may be far above the longest sequence.  Where it decides, that is, where sequences of equal length would not do (or one
// of max_seqlen among them might be too long), and the caller has given no host copy of cu_seqlens, both kernels are launched and the
// builders of their lists, who see the lengths, leave one of them empty (`pick` of a SchedView); that launch takes 4-9 us.  Backward, 32768 tokens
// in sequences of 128 under a bound of 8192, 32 heads: narrow 933, wide 1123, now 939; 49152 of 300 under 49152, 8 heads 468, 518, 477; exact
// bounds: 32768 tokens of Pareto lengths, 32 heads, d = 64 1062, 1026, 1026; 24000 of log-normal lengths, 10 heads 692, 669, 673.
enum { kKvNarrow = 0, kKvWide = 1, kKvByLengths = 2 };
int wide_kv(int T, int nseq, int max_seqlen, const int32_t* cu_host, int hq, int hkv, int head_dim, int wgs, long long* min_squares) {
    const bool four = hq / hkv >= 4;
    const double per_wg = (double)T / kKwBN * hkv / wgs, few = 1 + (four ? 1.4 : 2.5) / per_wg;       // items for each workgroup, about
    const double need = head_dim == 64 ? 400 * few : (four ? 600 : 1100) * (per_wg < 4 ? few : 1);
    *min_squares = (long long)(need * T);
    if (hkv >= 3 * kQueues && per_wg < (head_dim == 64 ? 2.4 : 3.1)) return kKvNarrow;
    const auto pays = [&](double squares, long long longest) { return wide_pays((unsigned long long)squares, longest, T, *min_squares, hkv, wgs); };
    const double m = nseq > 1 ? nseq - 1 : 1, rest = T - max_seqlen;
    if (!pays((double)max_seqlen * max_seqlen + rest * rest / m, max_seqlen)) return kKvNarrow;
    if (pays((double)T * T / nseq, max_seqlen)) return kKvWide;
    if (!cu_host) return kKvByLengths;
    double squares = 0;
    int longest = 0;
    for (int i = 0; i < nseq; ++i) {
        const int L = cu_host[i + 1] - cu_host[i];
        squares += (double)L * L;
        longest = L > longest ? L : longest;
    }
    return pays(squares, longest) ? kKvWide : kKvNarrow;
}
int item_heads(int split) { return split == 2 ? 4 : 1; }
// Form 3, of the forward only: 64 rows of one head, the waves sharing them (hyd_fwd_coop.h).
int form_shift(int split) { return split == 3 ? 2 : split; }      // rows of an item: 256 >> shift
// tiles of num_seqs sequences that hold T tokens, at most
long long most_items(int T, int nseq, int tile) { return ((long long)T + (long long)nseq * (tile - 1)) / tile; }
// The forward's size does not depend on the heads: one workspace serves layers of different head counts.
WsLayout fwd_layout(int T, int nseq, int hq, int hkv, int head_dim, hyd_dtype dt, bool compact) {
    WsLayout w = ws_layout(T, nseq, tile_q(dt), tile_q(dt), dt != HYD_BF16 || compact ? 0 : 2, hq, hkv, head_dim, dt, false, compact);
    if (!compact) {
        SchedLayout v;
        size_t most = sched_layout(v, 0, T, nseq, tile_q(dt), 0, false);
        if (dt == HYD_BF16) most = sched_layout(v, most, T, nseq, tile_q(dt) >> 2, 2, true);
        w.need = w.total = most + align_up(sizeof(double) * kRopeTabEntries);
    }
    return w;
}
WsLayout bwd_layout(int T, int nseq, int hq, int hkv, int head_dim, hyd_dtype dt, size_t bytes = 0) {
    return ws_layout(T, nseq, tile_kv(dt), tile_q(dt), finest_split(dt, hq, hkv, false), hq, hkv, head_dim, dt, true, false, bytes);
}

bool head_dim_ok(hyd_dtype dt, int d) { (void)dt; return d == 64 || d == 128; }

// Spread of (item, head) pairs over the 8 queues: whole KV groups per queue when the KV heads
// divide over the queues, else single heads, else items striped with all heads in every queue.
// `hq` counts the query heads in units of an item's heads.
HeadMap head_map_q(int hq, int hkv, int grid) {
    HeadMap hm;
    hm.grid = grid;
    hm.heads = hq;
    if (hkv % kQueues == 0) { hm.striped = 0; hm.hpq = hq / kQueues; hm.group = hq / hkv; }
    else if (hq % kQueues == 0) { hm.striped = 0; hm.hpq = hq / kQueues; hm.group = 1; }
    else { hm.striped = 1; hm.hpq = hq; hm.group = 1; }
    return hm;
}
HeadMap head_map_kv(int hkv, int grid) {
    HeadMap hm;
    hm.grid = grid;
    hm.heads = hkv;
    if (hkv % kQueues == 0) { hm.striped = 0; hm.hpq = hkv / kQueues; hm.group = 1; }
    else { hm.striped = 1; hm.hpq = hkv; hm.group = 1; }
    return hm;
}

hyd_status validate_common(const int32_t* cu, int num_seqs, const int32_t* cu_host, int T,
                           int max_seqlen, int hq, int hkv, int head_dim, hyd_dtype dt,
                           const void* ws, size_t ws_bytes, bool bwd, bool compact = false, bool own = false) {
    if (dt != HYD_BF16 && dt != HYD_FP32) return HYD_ERR_DTYPE;
    if (T < 0 || num_seqs < 0 || max_seqlen < 0) return HYD_ERR_SHAPE;
    if (num_seqs == 0 && T != 0) return HYD_ERR_SHAPE;
    if (hq <= 0 || hkv <= 0 || hq % hkv != 0) return HYD_ERR_HEADS;
    if (!head_dim_ok(dt, head_dim)) return HYD_ERR_HEADDIM;
    if (T == 0 || num_seqs == 0) return HYD_OK;
    if (!cu) return HYD_ERR_NULL;
    if (max_seqlen > T || max_seqlen < 1) return HYD_ERR_SHAPE;
    // a sequence must fit the 32-bit range of a buffer resource based at its first row
    if ((unsigned long long)max_seqlen * (unsigned long long)hq * (unsigned long long)head_dim *
            (dt == HYD_BF16 ? 2ull : 4ull) >= (dt == HYD_BF16 && head_dim == 64 ? (1ull << 31) : (1ull << 32)))
        return HYD_ERR_SHAPE;
    if (cu_host) {
        if (cu_host[0] != 0 || cu_host[num_seqs] != T) return HYD_ERR_SEQLENS;
        int longest = 0;
        for (int s = 0; s < num_seqs; ++s) {
            const int L = cu_host[s + 1] - cu_host[s];
            if (L < 0) return HYD_ERR_SEQLENS;
            if (L > longest) longest = L;
        }
        if (longest > max_seqlen) return HYD_ERR_SHAPE;
    }
    const WsLayout w = bwd ? bwd_layout(T, num_seqs, hq, hkv, head_dim, dt) : fwd_layout(T, num_seqs, hq, hkv, head_dim, dt, compact);
    const size_t need = own ? w.used : w.need;             // own: the library's array, made for this call
    if (!ws || ((uintptr_t)ws % kAlign) != 0 || ws_bytes < need) return HYD_ERR_WORKSPACE;
    return HYD_OK;
}

// Range variants: begins must fall on the coarsest tile boundary of the three kernels, ends
// either there or at / past the end of the sequence (then the sequence's length caps them).
static_assert(HYD_RANGE_ALIGN % kFwdBM == 0 && HYD_RANGE_ALIGN % kDqBM == 0 && HYD_RANGE_ALIGN % kKvBN == 0 &&
              HYD_RANGE_ALIGN % kFwdBN == 0 && HYD_RANGE_ALIGN % kDqBN == 0 && HYD_RANGE_ALIGN % kKvBM == 0,
              "range granule must be a multiple of every tile size");

hyd_status validate_ranges(const int32_t* ranges, const int32_t* ranges_host, const int32_t* cu_host,
                           int num_seqs, int max_seqlen, hyd_dtype dt) {
    if (dt != HYD_BF16) return HYD_ERR_DTYPE;
    if (num_seqs == 0) return HYD_OK;
    if (!ranges) return HYD_ERR_NULL;
    if (!ranges_host) return HYD_OK;
    for (int s = 0; s < num_seqs; ++s) {
        const int32_t* r = ranges_host + 4 * s;
        const int L = cu_host ? cu_host[s + 1] - cu_host[s] : max_seqlen;
        for (int e = 0; e < 2; ++e) {
            const int b = r[2 * e], en = r[2 * e + 1];
            if (b < 0 || b % HYD_RANGE_ALIGN != 0 || en < b) return HYD_ERR_RANGE;
            if (en % HYD_RANGE_ALIGN != 0 && en < L) return HYD_ERR_RANGE;
        }
    }
    return HYD_OK;
}

// ---- library-owned scratch of the entry point that allocates nothing ---------------------------
// Holds the forward's workspace (one schedule) for callers that cannot provide one.  Every GPU the
// library runs on keeps its own copy of this array until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress: the address kernels and memory calls use
// is DeviceInfo::scratch, looked up once per device.
constexpr size_t kScratchBytes = 2u << 20;
// (the cursors, 256 bytes apart, come on top of what callers size their batches for)
constexpr size_t kScratchAll = kScratchBytes + sizeof(int) * kQueues * kCursorStride;
static __device__ __align__(256) unsigned char scratch[kScratchAll];

// ---- per-device state -------------------------------------------------------------------------
struct DeviceInfo {
    bool ready = false, ok = false;
    int cus = 0;
    int occ_fwd = 1, occ_dq = 1, occ_kv = 1;
    int occ_f32[2][3] = {};           // [head_dim == 128][fwd, dQ, dK/dV]
    void* scratch = nullptr;          // this device's copy of the array above
};
DeviceInfo g_dev[64];
std::mutex g_dev_mutex;       // first use of a device from several host threads at once

template <typename K>
bool prep_kernel(K kernel, int threads, int lds, int* occ) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return false;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds) != hipSuccess) return false;
    if (occ) *occ = n < 1 ? 1 : n;
    return true;
}

template <int D>
bool prep_f32(int* occ) {
    return prep_kernel(hyd_fwd_fp32_kernel<D>, 64 * kF32Waves, f32_lds<D>(), occ) &&
           prep_kernel(hyd_bwd_dq_fp32_kernel<D>, 64 * kF32Waves, f32_lds<D>(), occ + 1) &&
           prep_kernel(hyd_fwd_self_fp32_kernel<D>, 64 * kF32Waves, f32_lds<D>(), nullptr) &&
           prep_kernel(hyd_bwd_dq_self_fp32_kernel<D>, 64 * kF32Waves, f32_lds<D>(), nullptr) &&
           prep_kernel(hyd_bwd_dkdv_fp32_kernel<D>, 64 * kF32KvWaves, f32_lds<D>(), occ + 2);
}

// [form of the items, then range variant][head_dim == 64]
typedef void (*FwdKernel)(FwdParams);
typedef void (*BwdKernel)(BwdParams, WorkList);
constexpr FwdKernel kFwdKernels[4][2] = {{hyd_fwd_bf16_kernel<false, 128, 0>, hyd_fwd_bf16_kernel<false, 64, 0>},
                                         {hyd_fwd_bf16_kernel<false, 128, 1>, hyd_fwd_bf16_kernel<false, 64, 1>},
                                         {hyd_fwd_bf16_kernel<false, 128, 2>, hyd_fwd_bf16_kernel<false, 64, 2>},
                                         {hyd_fwd_bf16_kernel<true, 128, 0>, hyd_fwd_bf16_kernel<true, 64, 0>}};
constexpr BwdKernel kDqKernels[4][2] = {{hyd_bwd_dq_bf16_kernel<false, 128, 0>, hyd_bwd_dq_bf16_kernel<false, 64, 0>},
                                        {hyd_bwd_dq_bf16_kernel<false, 128, 1>, hyd_bwd_dq_bf16_kernel<false, 64, 1>},
                                        {hyd_bwd_dq_bf16_kernel<false, 128, 2>, hyd_bwd_dq_bf16_kernel<false, 64, 2>},
                                        {hyd_bwd_dq_bf16_kernel<true, 128, 0>, hyd_bwd_dq_bf16_kernel<true, 64, 0>}};

typedef void (*FwdSelfKernel)(FwdParams, SelfSchedule);
constexpr FwdSelfKernel kFwdSelfKernels[2][2] = {{hyd_fwd_bf16_kernel<false, 128, 0, SelfSchedule>, hyd_fwd_bf16_kernel<false, 64, 0, SelfSchedule>},      // [half tiles][head_dim == 64]
                                                 {hyd_fwd_bf16_kernel<false, 128, 1, SelfSchedule>, hyd_fwd_bf16_kernel<false, 64, 1, SelfSchedule>}};
typedef void (*BothKernel)(BwdParams, WorkList, WorkList, int);
constexpr BothKernel kBothKernels[3][2] = {{hyd_bwd_both_bf16_kernel<128, 0>, hyd_bwd_both_bf16_kernel<64, 0>},
                                           {hyd_bwd_both_bf16_kernel<128, 1>, hyd_bwd_both_bf16_kernel<64, 1>},
                                           {hyd_bwd_both_bf16_kernel<128, 2>, hyd_bwd_both_bf16_kernel<64, 2>}};

hyd_status device_info(DeviceInfo** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return HYD_ERR_LAUNCH;
    if (dev < 0 || dev >= 64) return HYD_ERR_LAUNCH;
    DeviceInfo& d = g_dev[dev];
    std::lock_guard<std::mutex> lock(g_dev_mutex);
    if (!d.ready) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return HYD_ERR_LAUNCH;
        d.ok = strncmp(prop.gcnArchName, "gfx950", 6) == 0;
        d.cus = prop.multiProcessorCount;
        if (d.ok) {
            for (int i = 0; i < 8; ++i)          // (the LDS of all variants allows one workgroup per CU)
                if (!prep_kernel(kFwdKernels[i / 2][i % 2], kFwdThreads, kFwdLds, &d.occ_fwd) ||
                    !prep_kernel(kDqKernels[i / 2][i % 2], kDqThreads, kDqLds, &d.occ_dq))
                    return HYD_ERR_LAUNCH;
            if (!prep_kernel(hyd_fwd_coop_bf16_kernel, kFwdThreads, kCoLds, nullptr) || !prep_kernel(hyd_fwd_coop_self_bf16_kernel, kFwdThreads, kCoLds, nullptr))
                return HYD_ERR_LAUNCH;
            for (int i = 0; i < 4; ++i)
                if (!prep_kernel(kFwdSelfKernels[i / 2][i % 2], kFwdThreads, kFwdSelfLds, nullptr)) return HYD_ERR_LAUNCH;
            for (int i = 0; i < 6; ++i)
                if (!prep_kernel(kBothKernels[i / 2][i % 2], kKvThreads, kBothLds, nullptr)) return HYD_ERR_LAUNCH;
            if (!prep_kernel(hyd_bwd_dkdv_bf16_kernel<false>, kKvThreads, kKvLds, &d.occ_kv) ||
                !prep_kernel(hyd_bwd_dkdv_bf16_kernel<true>, kKvThreads, kKvLds, nullptr) ||
                !prep_kernel(hyd_bwd_dkdv_bf16_kernel<false, 64>, kKvThreads, kKvLds, nullptr) ||
                !prep_kernel(hyd_bwd_dkdv_bf16_kernel<true, 64>, kKvThreads, kKvLds, nullptr) ||
                !prep_kernel(hyd_bwd_dkdv_wide_bf16_kernel<128>, kKwThreads, kKwLds, nullptr) ||
                !prep_kernel(hyd_bwd_dkdv_wide_bf16_kernel<64>, kKwThreads, kKwLds, nullptr) ||
                !prep_f32<64>(d.occ_f32[0]) || !prep_f32<128>(d.occ_f32[1]))
                return HYD_ERR_LAUNCH;
            void* sp = nullptr;
            if (hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) != hipSuccess || !sp) return HYD_ERR_LAUNCH;
            d.scratch = sp;
        }
        d.ready = true;
    }
    if (!d.ok) return HYD_ERR_ARCH;
    *out = &d;
    return HYD_OK;
}

// ---- benchmark hooks --------------------------------------------------------------------------
struct TimedKernel { const char* name; hipEvent_t e0, e1; };
thread_local bool t_timing = false;
thread_local std::vector<TimedKernel> t_timed;
thread_local WgTrace t_trace = {nullptr, 0};

void timed_clear() {
    for (auto& t : t_timed) { (void)hipEventDestroy(t.e0); (void)hipEventDestroy(t.e1); }
    t_timed.clear();
}

constexpr size_t kMaxTimed = 8192;      // launches recorded between two reads of the list

struct KernelTimer {       // brackets one launch with events when timing is on
    hipStream_t st; bool on; TimedKernel tk;
    KernelTimer(const char* name, hipStream_t s) : st(s), on(t_timing && t_timed.size() < kMaxTimed) {
        tk.name = name;
        if (on) {
            on = hipEventCreate(&tk.e0) == hipSuccess && hipEventCreate(&tk.e1) == hipSuccess;
            if (on) (void)hipEventRecord(tk.e0, st);
        }
    }
    ~KernelTimer() {
        if (on) { (void)hipEventRecord(tk.e1, st); t_timed.push_back(tk); }
    }
};

// View of a schedule of `tile` rows (a 2^split-th of the kernel's tile); its level count is bounded by the caller's max_seqlen.
// `heads` work items per record are shared by `wgs` workgroups.  Sequences are grouped up to
// 1024 bf16 (512 fp32) rows, 512 KB of K and V for a head, unless four or more query heads share
// a KV head: their workgroups share its stream already, and the list's own order is balanced best.
SchedView make_view(char* ws, const SchedLayout& v, int tile, int split, int max_seqlen, hyd_dtype dt, int heads, int wgs, bool grouped_heads, int rec_heads = 1) {
    SchedView sv;
    sv.hdr = reinterpret_cast<int*>(ws + v.hdr);
    sv.lev = reinterpret_cast<int*>(ws + v.lev);
    sv.order = reinterpret_cast<int*>(ws + v.order);
    sv.items = reinterpret_cast<int*>(ws + v.items);
    const int by_len = levels(max_seqlen, tile, split);
    sv.n_lev = by_len < v.n_lev ? by_len : v.n_lev;
    sv.max_items = v.max_items;
    sv.exec = reinterpret_cast<int*>(ws + v.exec);
    sv.group_max = v.exec == v.items || grouped_heads ? 0 : (dt == HYD_BF16 ? 1024 : 512) / tile;
    sv.group_share = (float)heads / (16.f * (float)wgs);
    sv.part_max = 1; sv.part_q = 1; sv.steps_per_level = 0;
    sv.other = 0; sv.rec_heads = rec_heads;
    sv.pick = 0; sv.pick_hkv = sv.pick_wgs = 1; sv.pick_squares = 0;
    return sv;
}

// Parts of the dK/dV items.  An item runs over the query tiles of its sequence for every head of the
// group in turn, so with few KV heads or few tokens the longest items last longer than all the work does
// spread over the workgroups.  The work is bounded from below by what the host knows (one sequence of
// max_seqlen tokens, the others of equal length): where the longest item is well above a workgroup's
// share of that, items are cut into parts of half a share, at least kPartSteps steps.  The fp32 sums
// of a part cost about as much as five steps, and the pass that adds them 7-20 us, which is why an item
// of less than two such parts, or less than 1.6 shares, stays whole (dK/dV in us, whole -> in parts with
// the adding pass: 4096 tokens in one sequence, 10 heads, 1.55 shares: 121 -> 139; 16384 tokens, 64/8
// heads, 1.05 shares: 1068 -> 1083).
// Measured (log-normal lengths, dK/dV + adding pass in us, before -> now): 8/1 heads, 8192 tokens 650 ->
// 123; 16/2 heads, 8192 tokens 666 -> 233, 32768 tokens 1428 -> 820; 8/1 heads, one sequence of 16384
// tokens 3070 -> 1262; 32/8 heads, 512 tokens 54 -> 41, 1024 tokens 98 -> 47, 2048 tokens 115 -> 78, 4096 tokens 307 -> 221,
// 8192 tokens 415 -> 406.  kPartSteps 12 / 16 / 24 / 40: 512 tokens 36 / 41 / 50 / 54, 1024 tokens 43 / 47 / 54 / 74, 2048 tokens 76 /
// 78 / 65 / 81; with 12 a batch of 8/8 heads and 2048 tokens is cut too, for nothing (37 -> 37).
void set_parts(SchedView& sv, int limit, int T, int nseq, int max_seqlen, int hq, int hkv, int wgs) {
    sv.steps_per_level = kKvBN / kKvBM * (hq / hkv);
    const double share = share_of_work(kKvBN, sv.steps_per_level, T, nseq, max_seqlen, hkv, wgs);
    const double longest = (double)sv.n_lev * sv.steps_per_level;
    const double q = steps_of_part(longest, share, limit);
    if (q == 0) return;
    sv.part_q = (int)ceil(q);
    sv.part_max = item_parts(sv.n_lev, sv.steps_per_level, sv.part_q, limit);
}

// Where dK/dV shares a launch with dQ: the workgroups that it has, one per item where there is room for all items, else four of
// seven (its share of the products);
int both_kv_workgroups(int cus, long long work_q) {
    const int n = cus * 4 / 7;
    return n < cus - work_q ? (int)(cus - work_q) : n;
}

// Items in other parts than those of set_parts, mostly finer, where dK/dV shares a launch with dQ and its longest item makes the launch: down
// to 4 steps, as fine as the parts still all start at once (a level in n parts of q steps: half a part more than its steps / q on average), and
// not finer than what the longest dQ item lasts (its tile of 64 keys counts 1.2 steps for 64 rows of four heads, half a step
// where four waves share 128 rows).  A step takes 0.6-0.85 us and the adding pass 5-6, so that cutting has to take 8 steps off.
// Backward in us, one sequence unless noted: 256 tokens, 8/1 heads 49.1 -> 28.8, 256, 32/8 heads 43.4 -> 32.0, 700, 32/8 54.0 -> 48.2, 900,
// 2/1 47.4 -> 35.9, 1500, 8 heads 61.4 -> 53.4, 3000 tokens of 64-1024, 8/1 56.9 -> 51.2.  Without the bound by room 3000 tokens, 8 heads
// 77.3 -> 80.6, 700, 32 heads 48.0 -> 58.1; without the one by dQ 2200, 2/1 heads 62.9 -> 65.1.
// Where those of set_parts are taken (dK/dV after dQ, before, now): 17000 tokens, 2/1 heads 682 / 916 / 615, 14000 480 / 553 / 449, 7000, 4/2
// 271 / 300 / 252, 20480 of log-normal lengths, 2/1 207 / 219 / 157, 10200, 4/2 133 / 143 / 104; always, 5120, 8/1 heads 250 -> 326, 5000, 4/1 135 -> 173.
void both_parts(SchedView& sv, int limit, int T, int nseq, int max_seqlen, int hq, int hkv, int cus, long long work_q, int split) {
    const double longest = (double)sv.n_lev * sv.steps_per_level, room = both_kv_workgroups(cus, work_q) - 0.5 * most_items(T, nseq, kKvBN) * hkv;
    if (limit <= 1 || room <= 0) return;
    const int others = nseq > 1 ? ((T - max_seqlen) / (nseq - 1) + kKvBN - 1) / kKvBN : 0;      // tiles of each, if alike
    const double steps = share_of_work(1, sv.steps_per_level, sv.n_lev + (nseq - 1) * others, nseq, sv.n_lev, hkv, 1);
    double q = fmax(fmax(kBothPartSteps, steps / room), max_seqlen / (split == 2 ? 54.0 : 128.0));
    q = fmax(q, longest / limit);
    if (sv.part_max > 1) {
        // Many items leave little room, and parts that all start at once are long then; those of set_parts, in turn, last about a
        // workgroup's share and half a part.  (With 4/5 against what the estimate leaves out.)
        const double again = fmax(steps / both_kv_workgroups(cus, work_q) + 0.5 * sv.part_q, max_seqlen / (split == 2 ? 54.0 : 128.0));
        if (again < 0.8 * q) return;
    }
    if (longest < q + kBothPartGain) return;
    sv.part_q = (int)ceil(q);
    sv.part_max = item_parts(sv.n_lev, sv.steps_per_level, sv.part_q, limit);
}

// Every (item, head) pair gets a workgroup of its own, and the lists theirs (see SelfSchedule): where all run at once, and up
// to 1.75 for each CU (1.5 if no sequence is long) where the launch lasts as long as its longest item (see query_split), or where two or
// three sequences of up to 2048 tokens hold them; they then come longest first.  Forward, list -> own items in us: one sequence of
// 1500 tokens, 32 heads (430 items) 32.3 -> 25.8; 10240 tokens of log-normal lengths, 5 heads (430) 67.8 -> 62.1; 6656 of 64-1024, 5 heads
// (320) 29.3 -> 23.9; 2040 in sequences of 2000, 32/8 heads (288 whole tiles) 58.2 -> 53.5.  Beyond that the hardware, which
// hands workgroups to the XCDs strictly in turn, balances the later ones badly (sequence by sequence, 8 heads: one sequence of 8000 tokens, 504
// items, 186 -> 196; 16000, 504 whole tiles, 449 -> 485).  fp32, d = 128, sequence by sequence: 2400 tokens of 64-1024, 8 heads 77.7 -> 69.2; 2400
// of equal lengths 53.7 -> 62.4, 5600, 4 heads 59 -> 89, so that none has more than one item per CU there.
bool self_schedule_ok(hyd_dtype dt, int nseq, long long work, int lists, bool uneven, int max_seqlen, int cus) {
    if (nseq > kSelfSeqs) return false;
    if (work + lists <= cus) return true;
    const bool few = nseq <= 3 && max_seqlen <= 2048;
    return dt == HYD_BF16 && (uneven || few) && 4 * work <= (max_seqlen > 1024 || few ? 7 : 6) * cus && max_seqlen <= 6144;
}
// Form 3 instead of half tiles where the launch starts with all of its items.  Those that come second cost what an item costs at
// least, 8 us (10 with rotary positions, whose angles the four waves of a row each form), and 128 keys of the longest item take 0.48 us
// less: up to 1.5 items for each CU pay from some 800 tokens on (1000 with rotary positions), up to 2 from 2048.  Forward, half tiles ->
// form 3 in us (in brackets its items), d = 128: one sequence of 256 tokens, 8 heads
// (32) 9.9 -> 9.5, 700, 32 heads (352) 17.5 -> 15.5, 1500, 8 heads (192) 29.7 -> 23.2, 3000, 8 heads (376) 52.4 -> 41.6, 4000 (504)
// 67.8 -> 64.4, 6000 (752) 103 -> 135; sequences of 64-1024: 2000 tokens, 8 heads (280) 16.8 -> 14.0, 3000 (416) 18.6 -> 20.2; of 146, 8
// heads (280) 8.5 -> 12.1, 410, 2 heads (336) 11.9 -> 12.7, 600, 3 heads (339) 16.9 -> 19.0, 773, 2 heads (340) 17.4 -> 15.8, 848, 10 heads
// (280) 19.8 -> 17.0; with rotary positions 81, 8 heads (336) 9.6 -> 15.8 (whole tiles from a list 15.2), 822, 5 heads (345) 21.6 -> 23.1, 950, 1 head
// (344) 21.5 -> 19.7.  (With d = 64, where the second product occupied two waves of four, 1500 tokens, 8 heads 19.1 -> 18.2, 700, 32
// heads 13.7 -> 14.0.)
// From a list only where an XCD keeps to few heads (see head_map_q), since 64 rows read a head's keys four times as often as 256, and from 3000
// tokens on, since half tiles need none there: one sequence, from a list: 25600 tokens, 1 head (400) 382 -> 330, 6528, 5 heads (510) 107 -> 111,
// 2880, 10 heads (450) 49.3 -> 58.1, 3264 (510) 60.4 -> 67.8; several up to 2712, 3 heads (501) 45.8 -> 51.2, 2499, 8 heads (496) 43.6 -> 46.7, 3094 (512)
// 51.4 -> 49.4.
int fwd_form(int split, int T, int nseq, int max_seqlen, int hq, int head_dim, bool rope, int cus) {
    if (split != 1 || head_dim != 128) return split;
    const long long items = most_items(T, nseq, 64) * hq;
    if (items + 2 <= cus) return 3;
    if (max_seqlen < (rope ? 1000 : 800)) return 1;
    if (2 * items <= 3 * cus) return 3;
    if (items > 2 * cus || max_seqlen < 2048) return 1;
    return self_schedule_ok(HYD_BF16, nseq, items, 2, true, max_seqlen, cus) || ((hq % kQueues == 0 || hq < 4) && max_seqlen >= 3000) ? 3 : 1;
}

SelfSchedule self_schedule(const int32_t* cu, int nseq, int T, int work, int lists, int heads, int tile, const SchedView& sv, int cus) {
    SelfSchedule ss;
    ss.cu = cu; ss.nseq = nseq; ss.T = T; ss.n_work = work; ss.heads = heads; ss.tile = tile; ss.n_lev = sv.n_lev;
    ss.by_level = work + lists > cus;
    ss.n_lists = 0; ss.log2_base = 0.0;
    return ss;
}
void add_list(SelfSchedule& ss, int tile, const SchedView& sv) { ss.tiles[ss.n_lists] = tile; ss.lists[ss.n_lists++] = sv; }

int persistent_grid(const DeviceInfo& d, int occ, long long work_upper_bound) {
    long long g = (long long)d.cus * occ;
    if (g > work_upper_bound) g = work_upper_bound;
    return g < 1 ? 1 : (int)g;
}

}  // namespace

extern "C" {

const char* hyd_status_string(hyd_status st) {
    switch (st) {
        case HYD_OK: return "HYD_OK";
        case HYD_ERR_NULL: return "HYD_ERR_NULL: a required pointer is NULL";
        case HYD_ERR_SHAPE: return "HYD_ERR_SHAPE: negative size or max_seqlen out of range";
        case HYD_ERR_DTYPE: return "HYD_ERR_DTYPE: unknown dtype";
        case HYD_ERR_HEADS: return "HYD_ERR_HEADS: hq and hkv must be positive with hq % hkv == 0";
        case HYD_ERR_HEADDIM: return "HYD_ERR_HEADDIM: head_dim must be 64 or 128";
        case HYD_ERR_SEQLENS: return "HYD_ERR_SEQLENS: cu_seqlens must start at 0, end at T and not decrease";
        case HYD_ERR_WORKSPACE: return "HYD_ERR_WORKSPACE: workspace NULL, misaligned or too small";
        case HYD_ERR_ARCH: return "HYD_ERR_ARCH: device is not gfx950";
        case HYD_ERR_LAUNCH: return "HYD_ERR_LAUNCH: HIP launch or query failed";
        case HYD_ERR_INFEASIBLE: return "HYD_ERR_INFEASIBLE: the planning constraints admit no solution";
        case HYD_ERR_RANGE: return "HYD_ERR_RANGE: a range begin is not a multiple of HYD_RANGE_ALIGN, or an end is neither that nor past the sequence";
    }
    return "unknown hyd_status";
}

size_t hyd_varlen_attn_workspace_bytes(int total_tokens, int num_seqs, int hq, int hkv, int head_dim,
                                       hyd_dtype dt, int is_bwd) {
    if (total_tokens < 0 || num_seqs < 0 || hq <= 0 || hkv <= 0 || hq % hkv != 0) return 0;
    if ((dt != HYD_BF16 && dt != HYD_FP32) || !head_dim_ok(dt, head_dim)) return 0;
    return (is_bwd ? bwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt)
                   : fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, false)).total;
}

}  // extern "C"

namespace {

// forward of the plain entry point (ranges == NULL) and of the range variant
// rope_base: 0 = no rotation, else the base of the rotary embedding applied to Q inside the kernels
hyd_status fwd_impl(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                    int num_seqs, const int32_t* cu_seqlens_host, const int32_t* ranges,
                    const int32_t* ranges_host, bool ranged, int total_tokens,
                    int max_seqlen, int hq, int hkv, int head_dim, float softmax_scale,
                    hyd_dtype dt, void* o, float* lse, void* workspace,
                    size_t workspace_bytes, void* hip_stream, float rope_base = 0.f, bool compact = false, bool own = false) {
    if (rope_base != 0.f && (dt != HYD_BF16 || !(rope_base > 1.f))) return dt != HYD_BF16 ? HYD_ERR_DTYPE : HYD_ERR_SHAPE;
    const hyd_status vs = validate_common(cu_seqlens, num_seqs, cu_seqlens_host, total_tokens, max_seqlen,
                                          hq, hkv, head_dim, dt, workspace, workspace_bytes, false, compact, own);
    if (vs != HYD_OK) return vs;
    if (ranged) {
        const hyd_status rs = validate_ranges(ranges, ranges_host, cu_seqlens_host, num_seqs, max_seqlen, dt);
        if (rs != HYD_OK) return rs;
    }
    if (total_tokens == 0 || num_seqs == 0) return HYD_OK;
    if (!q || !k || !v || !o || !lse) return HYD_ERR_NULL;

    DeviceInfo* dev = nullptr;
    const hyd_status ds = device_info(&dev);
    if (ds != HYD_OK) return ds;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    const int split = ranged ? 0 : fwd_form(query_split(dt, total_tokens, num_seqs, max_seqlen, hq, hkv, compact), total_tokens, num_seqs, max_seqlen, hq, head_dim, rope_base != 0.f, dev->cus), shift = form_shift(split);
    const int tile = tile_q(dt), units = hq / item_heads(split);
    const WsLayout w = fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, compact);
    const int occ = dt == HYD_BF16 ? dev->occ_fwd : dev->occ_f32[head_dim == 128][0];
    // where items are not whole tiles, the list of whole tiles is built too, next to the one that is
    // handed out (hyd_varlen_attn_schedule_layout shows the first and its header leads to the second)
    const bool grouped = hq >= 4 * hkv;
    SchedView sv_whole = make_view(static_cast<char*>(workspace), w.sched[0], tile, 0, max_seqlen, dt, units, dev->cus * occ, grouped);
    if (split) sv_whole.other = (int)(w.split.hdr - w.sched[0].hdr);
    const SchedView sv = split ? make_view(static_cast<char*>(workspace), w.split, 256 >> shift, shift, max_seqlen, dt, units, dev->cus * occ, grouped, item_heads(split)) : sv_whole;
    double* rope_tab = rope_base != 0.f ? reinterpret_cast<double*>(static_cast<char*>(workspace) + w.rope_tab) : nullptr;
    const long long work = (long long)sv.max_items * units, self_work = most_items(total_tokens, num_seqs, tile >> shift) * units;
    const bool self = !ranged && split != 2 && self_schedule_ok(dt, num_seqs, self_work, split ? 2 : 1, split != 0, max_seqlen, dev->cus);
    SelfSchedule ss;
    if (self) {
        ss = self_schedule(cu_seqlens, num_seqs, total_tokens, (int)self_work, split ? 2 : 1, units, tile >> shift, sv, dev->cus);
        add_list(ss, tile, sv_whole);
        if (split) add_list(ss, tile >> shift, sv);
        ss.log2_base = rope_base != 0.f ? log2((double)rope_base) : 0.0;
    } else {
        KernelTimer kt("schedule_prelude", st);
        hipLaunchKernelGGL(hyd_schedule_prelude, dim3(split ? 2 : 1), dim3(kPreludeThreads), schedule_lds(sv_whole.n_lev, sv.n_lev), st, cu_seqlens, num_seqs,
                           total_tokens, tile, sv_whole, tile >> shift, sv,
                           rope_tab, head_dim / 2, rope_base != 0.f ? log2((double)rope_base) : 0.0);
    }
    if (dt == HYD_BF16) {
        FwdParams p;
        p.q = static_cast<const uint16_t*>(q); p.k = static_cast<const uint16_t*>(k);
        p.v = static_cast<const uint16_t*>(v); p.o = static_cast<uint16_t*>(o); p.lse = lse;
        p.T = total_tokens; p.hq = hq; p.hkv = hkv;
        p.scale_log2 = softmax_scale * kLog2e;
        p.hdr = sv.hdr; p.cursors = sv.hdr + kHdrCursor; p.items = sv.exec; p.tr = t_trace;
        p.ranges = ranged ? ranges : nullptr;
        p.rope_tab = rope_tab;
        const dim3 grid(persistent_grid(*dev, occ, work));
        p.hm = head_map_q(units, hkv, grid.x);
        KernelTimer kt(ranged ? "fwd_range_bf16" : "fwd_bf16", st);
        if (split == 3 && self) hipLaunchKernelGGL(hyd_fwd_coop_self_bf16_kernel, dim3(ss.n_work + ss.n_lists), dim3(kFwdThreads), kCoLds, st, p, ss);
        else if (split == 3) hipLaunchKernelGGL(hyd_fwd_coop_bf16_kernel, grid, dim3(kFwdThreads), kCoLds, st, p);
        else if (self) hipLaunchKernelGGL(kFwdSelfKernels[split][head_dim == 64], dim3(ss.n_work + ss.n_lists), dim3(kFwdThreads), kFwdSelfLds, st, p, ss);
        else hipLaunchKernelGGL(kFwdKernels[ranged ? 3 : split][head_dim == 64], grid, dim3(kFwdThreads), kFwdLds, st, p);
    } else {
        F32Params p;
        memset(&p, 0, sizeof(p));
        p.q = static_cast<const float*>(q); p.k = static_cast<const float*>(k);
        p.v = static_cast<const float*>(v); p.o_out = static_cast<float*>(o); p.lse_out = lse;
        p.T = total_tokens; p.hq = hq; p.hkv = hkv; p.scale = softmax_scale;
        p.hdr = sv.hdr; p.cursors = sv.hdr + kHdrCursor; p.items = sv.exec; p.tr = t_trace;
        const dim3 grid(persistent_grid(*dev, occ, work));
        p.hm = head_map_q(hq, hkv, grid.x);
        KernelTimer kt("fwd_fp32", st);
        const auto self_kernel = head_dim == 64 ? hyd_fwd_self_fp32_kernel<64> : hyd_fwd_self_fp32_kernel<128>;
        if (self) hipLaunchKernelGGL(self_kernel, dim3(ss.n_work + ss.n_lists), dim3(64 * kF32Waves), head_dim == 64 ? f32_lds<64>() : f32_lds<128>(), st, p, ss);
        else if (head_dim == 64) hipLaunchKernelGGL(hyd_fwd_fp32_kernel<64>, grid, dim3(64 * kF32Waves), f32_lds<64>(), st, p);
        else hipLaunchKernelGGL(hyd_fwd_fp32_kernel<128>, grid, dim3(64 * kF32Waves), f32_lds<128>(), st, p);
    }
    return hipGetLastError() == hipSuccess ? HYD_OK : HYD_ERR_LAUNCH;
}

// backward of the plain entry point (ranges == NULL) and of the range variant
hyd_status bwd_impl(const void* q, const void* k, const void* v, const void* o, const float* lse,
                    const void* d_o, const int32_t* cu_seqlens, int num_seqs,
                    const int32_t* cu_seqlens_host, const int32_t* ranges, const int32_t* ranges_host,
                    bool ranged, int total_tokens, int max_seqlen, int hq,
                    int hkv, int head_dim, float softmax_scale, hyd_dtype dt, void* dq, void* dk,
                    void* dv, void* workspace, size_t workspace_bytes, void* hip_stream, float rope_base = 0.f) {
    if (rope_base != 0.f && (dt != HYD_BF16 || !(rope_base > 1.f))) return dt != HYD_BF16 ? HYD_ERR_DTYPE : HYD_ERR_SHAPE;
    const hyd_status vs = validate_common(cu_seqlens, num_seqs, cu_seqlens_host, total_tokens, max_seqlen,
                                          hq, hkv, head_dim, dt, workspace, workspace_bytes, true);
    if (vs != HYD_OK) return vs;
    if (ranged) {
        const hyd_status rs = validate_ranges(ranges, ranges_host, cu_seqlens_host, num_seqs, max_seqlen, dt);
        if (rs != HYD_OK) return rs;
    }
    if (total_tokens == 0 || num_seqs == 0) return HYD_OK;
    if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv) return HYD_ERR_NULL;

    DeviceInfo* dev = nullptr;
    const hyd_status ds = device_info(&dev);
    if (ds != HYD_OK) return ds;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    const WsLayout w = bwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, workspace_bytes);
    char* ws = static_cast<char*>(workspace);
    const int occ_q = dt == HYD_BF16 ? dev->occ_dq : dev->occ_f32[head_dim == 128][1];
    const int occ_kv = dt == HYD_BF16 ? dev->occ_kv : dev->occ_f32[head_dim == 128][2];
    const int split = ranged ? 0 : query_split(dt, total_tokens, num_seqs, max_seqlen, hq, hkv, false);
    const int units = hq / item_heads(split);
    const bool grouped = hq >= 4 * hkv;
    SchedView sv_kv = make_view(ws, w.sched[0], tile_kv(dt), 0, max_seqlen, dt, hkv, dev->cus * occ_kv, grouped);
    const bool both = dt == HYD_BF16 && !ranged && rope_base == 0.f && both_ok(total_tokens, num_seqs, max_seqlen, hq, hkv, dev->cus);
    SchedView sv_whole = make_view(ws, w.sched[1], tile_q(dt), 0, max_seqlen, dt, units, dev->cus * occ_q, grouped);
    if (split) sv_whole.other = (int)(w.split.hdr - w.sched[1].hdr);
    const SchedView sv_q = split ? make_view(ws, w.split, 256 >> split, split, max_seqlen, dt, units, dev->cus * occ_q, grouped, item_heads(split)) : sv_whole;
    const long long work_q = (long long)sv_q.max_items * units;
    if (dt == HYD_BF16) set_parts(sv_kv, w.part_max, total_tokens, num_seqs, max_seqlen, hq, hkv, dev->cus * occ_kv);
    if (both) both_parts(sv_kv, w.part_max, total_tokens, num_seqs, max_seqlen, hq, hkv, dev->cus, work_q, split);
    long long min_squares = 0;
    const int wide = dt == HYD_BF16 && !ranged && !both && sv_kv.part_max == 1 ?
                     wide_kv(total_tokens, num_seqs, max_seqlen, cu_seqlens_host, hq, hkv, head_dim, dev->cus, &min_squares) : kKvNarrow;
    SchedView sv_wide = wide ? make_view(ws, w.wide, kKwBN, 0, max_seqlen, dt, hkv, dev->cus, grouped) : sv_kv;
    if (wide) sv_kv.other = (int)(w.wide.hdr - w.sched[0].hdr);
    if (wide == kKvByLengths) {
        sv_kv.pick = -1; sv_wide.pick = 1;
        sv_kv.pick_hkv = sv_wide.pick_hkv = hkv; sv_kv.pick_wgs = sv_wide.pick_wgs = dev->cus; sv_kv.pick_squares = sv_wide.pick_squares = min_squares;
    }
    float* Dvec = reinterpret_cast<float*>(ws + w.stat[0]);
    double* rope_tab = rope_base != 0.f ? reinterpret_cast<double*>(ws + w.rope_tab) : nullptr;
    const long long work_kv = (long long)sv_kv.max_items * sv_kv.part_max * hkv;
    if (dt == HYD_BF16) {
        BwdScratch sc;
        sc.Dq = Dvec;
        sc.kqmul = reinterpret_cast<float*>(ws + w.stat[1]);
        sc.lse2 = reinterpret_cast<float*>(ws + w.stat[2]);
        sc.Dkv = reinterpret_cast<float*>(ws + w.stat[3]);
        sc.q16 = reinterpret_cast<uint16_t*>(ws + w.q16);
        sc.do16 = reinterpret_cast<uint16_t*>(ws + w.do16);
        sc.k16 = reinterpret_cast<uint16_t*>(ws + w.k16);
        // item lists of both tile kernels and the row statistics in one launch
        {
            PrepParams pp;
            pp.o = static_cast<const uint16_t*>(o); pp.d_o = static_cast<const uint16_t*>(d_o); pp.lse = lse; pp.k = static_cast<const uint16_t*>(k);
            pp.q = static_cast<const uint16_t*>(q);
            pp.T = total_tokens; pp.hq = hq; pp.hkv = hkv; pp.tok = prep_tokens(total_tokens, hq);
            sc.absmax = reinterpret_cast<uint32_t*>(ws + w.absmax);
            sc.n_absmax = prep_workgroups(total_tokens, pp.tok);
            pp.sc = sc;
            pp.cu = cu_seqlens; pp.nseq = num_seqs;
            pp.ranges = ranged ? ranges : nullptr;
            pp.n_sched = 0;
            const auto add_list = [&](int tile, const SchedView& sv) { pp.tile[pp.n_sched] = tile; pp.sv[pp.n_sched++] = sv; };
            add_list(tile_kv(dt), sv_kv);
            add_list(tile_q(dt), sv_whole);
            if (split) add_list(tile_q(dt) >> split, sv_q);
            if (wide) add_list(kKwBN, sv_wide);
            pp.rope_tab = rope_tab; pp.log2_base = rope_tab ? log2((double)rope_base) : 0.0;
            const dim3 grid((unsigned)(pp.n_sched + sc.n_absmax)), block(kPrepThreads);
            const size_t lds = prep_lds(hq, pp.tok, schedule_lds(sv_kv.n_lev, sv_whole.n_lev, sv_q.n_lev, sv_wide.n_lev));
            KernelTimer kt("bwd_prep_bf16", st);
            const auto kernel = both ? (head_dim == 64 ? hyd_bwd_prep_bf16_kernel<false, 64, true> : hyd_bwd_prep_bf16_kernel<false, 128, true>)
                : ranged ? (head_dim == 64 ? hyd_bwd_prep_bf16_kernel<true, 64> : hyd_bwd_prep_bf16_kernel<true, 128>)
                         : (head_dim == 64 ? hyd_bwd_prep_bf16_kernel<false, 64> : hyd_bwd_prep_bf16_kernel<false, 128>);
            hipLaunchKernelGGL(kernel, grid, block, lds, st, pp);
        }
        BwdParams p;
        p.q = static_cast<const uint16_t*>(q); p.v = static_cast<const uint16_t*>(v); p.d_o = static_cast<const uint16_t*>(d_o);
        p.sc = sc;
        p.dq = static_cast<uint16_t*>(dq); p.dk = static_cast<uint16_t*>(dk); p.dv = static_cast<uint16_t*>(dv);
        p.T = total_tokens; p.hq = hq; p.hkv = hkv;
        p.scale = softmax_scale; p.scale_log2 = softmax_scale * kLog2e;
        p.tr = t_trace;
        p.ranges = ranged ? ranges : nullptr;
        p.rope_tab = rope_tab;
        p.part = reinterpret_cast<float*>(ws + w.need); p.part_max = sv_kv.part_max;
        const int grid_q = persistent_grid(*dev, occ_q, work_q), grid_kv = persistent_grid(*dev, occ_kv, work_kv);
        WorkList lq{sv_q.hdr, sv_q.hdr + kHdrCursor, sv_q.exec, head_map_q(units, hkv, grid_q)};
        WorkList lkv{sv_kv.hdr + kHdrExec, sv_kv.hdr + kHdrCursor, sv_kv.exec, head_map_kv(hkv, grid_kv)};
        if (both) {
            int n_kv = both_kv_workgroups(dev->cus, work_q);
            if (n_kv > work_kv) n_kv = (int)work_kv;
            n_kv = (n_kv + kQueues - 1) / kQueues * kQueues;           // queue by XCD on both sides
            int n_q = dev->cus - n_kv;
            if (n_q > work_q) n_q = (int)work_q;
            if (n_q < 0) n_q = 0;
            lkv.hm.grid = n_kv; lq.hm.grid = n_q;
            KernelTimer kt("bwd_both_bf16", st);
            hipLaunchKernelGGL(kBothKernels[split][head_dim == 64], dim3(n_kv + n_q), dim3(kKvThreads), kBothLds, st, p, lkv, lq, n_kv);
        } else {
            {   // dQ first: it also writes the fp16 copies of Q and dO that dK/dV streams
                KernelTimer kt(ranged ? "bwd_dq_range_bf16" : "bwd_dq_bf16", st);
                hipLaunchKernelGGL(kDqKernels[ranged ? 3 : split][head_dim == 64], dim3(grid_q), dim3(kDqThreads), kDqLds, st, p, lq);
            }
            KernelTimer kt(ranged ? "bwd_dkdv_range_bf16" : "bwd_dkdv_bf16", st);
            const BwdKernel kernel = ranged ? (head_dim == 64 ? hyd_bwd_dkdv_bf16_kernel<true, 64> : hyd_bwd_dkdv_bf16_kernel<true, 128>)
                                            : (head_dim == 64 ? hyd_bwd_dkdv_bf16_kernel<false, 64> : hyd_bwd_dkdv_bf16_kernel<false, 128>);
            if (wide) {
                const int grid = persistent_grid(*dev, 1, (long long)sv_wide.max_items * hkv);
                const WorkList list{sv_wide.hdr + kHdrExec, sv_wide.hdr + kHdrCursor, sv_wide.exec, head_map_kv(hkv, grid)};
                hipLaunchKernelGGL(head_dim == 64 ? hyd_bwd_dkdv_wide_bf16_kernel<64> : hyd_bwd_dkdv_wide_bf16_kernel<128>, dim3(grid), dim3(kKwThreads), kKwLds, st, p, list);
            }
            if (wide != kKvWide) hipLaunchKernelGGL(kernel, dim3(grid_kv), dim3(kKvThreads), kKvLds, st, p, lkv);
        }
        if (sv_kv.part_max > 1) {
            SumParams sp;
            sp.part = p.part; sp.dk = p.dk; sp.dv = p.dv; sp.T = total_tokens; sp.hkv = hkv;
            sp.part_max = sv_kv.part_max; sp.part_q = sv_kv.part_q; sp.steps_per_level = sv_kv.steps_per_level;
            sp.hdr = sv_kv.hdr; sp.items = sv_kv.items; sp.ranges = p.ranges;
            // items in parts are the first of the list: those of levels above `low`, of sequences longer than low tiles
            const long long low = sp.part_q / sp.steps_per_level, tiles = total_tokens / kKvBN + 1;
            const long long bound = low > 0 ? tiles + tiles / low + 1 : sv_kv.max_items;
            const dim3 grid((unsigned)(bound < sv_kv.max_items ? bound : sv_kv.max_items), (unsigned)hkv, 2 * kKvBN / kSumRows);
            KernelTimer kt("bwd_sum_parts", st);
            if (head_dim == 64) hipLaunchKernelGGL(hyd_bwd_sum_parts_kernel<64>, grid, dim3(kSumThreads), 0, st, sp);
            else hipLaunchKernelGGL(hyd_bwd_sum_parts_kernel<128>, grid, dim3(kSumThreads), 0, st, sp);
        }
    } else {
        F32Params p;
        memset(&p, 0, sizeof(p));
        p.q = static_cast<const float*>(q); p.k = static_cast<const float*>(k);
        p.v = static_cast<const float*>(v); p.o = static_cast<const float*>(o);
        p.d_o = static_cast<const float*>(d_o); p.lse_in = lse; p.D = Dvec;
        p.dq = static_cast<float*>(dq); p.dk = static_cast<float*>(dk); p.dv = static_cast<float*>(dv);
        p.T = total_tokens; p.hq = hq; p.hkv = hkv; p.scale = softmax_scale;
        p.tr = t_trace;
        const bool short_rows = max_seqlen <= kF32Short;
        const long long self_work = most_items(total_tokens, num_seqs, tile_q(dt)) * hq;
        const bool self = !short_rows && self_schedule_ok(dt, num_seqs, self_work, 2, false, max_seqlen, dev->cus);
        if (!self) {   // one launch builds both item lists, one workgroup each
            KernelTimer kt("schedule_prelude", st);
            hipLaunchKernelGGL(hyd_schedule_prelude, dim3(w.n_sched), dim3(kPreludeThreads), schedule_lds(sv_kv.n_lev, sv_q.n_lev), st, cu_seqlens,
                               num_seqs, total_tokens, tile_kv(dt), sv_kv, tile_q(dt), sv_q, nullptr, 0, 0.0);
        }
        const dim3 grid_q(persistent_grid(*dev, occ_q, work_q)), grid_kv(persistent_grid(*dev, occ_kv, work_kv));
        // dQ first: it also writes the row sums D that dK/dV reads
        {
            p.hdr = sv_q.hdr; p.items = sv_q.exec; p.cursors = sv_q.hdr + kHdrCursor; p.hm = head_map_q(hq, hkv, grid_q.x);
            KernelTimer kt("bwd_dq_fp32", st);
            if (self) {
                SelfSchedule ss = self_schedule(cu_seqlens, num_seqs, total_tokens, (int)self_work, 2, hq, tile_q(dt), sv_q, dev->cus);
                add_list(ss, tile_kv(dt), sv_kv);
                add_list(ss, tile_q(dt), sv_q);
                const auto self_kernel = head_dim == 64 ? hyd_bwd_dq_self_fp32_kernel<64> : hyd_bwd_dq_self_fp32_kernel<128>;
                hipLaunchKernelGGL(self_kernel, dim3(ss.n_work + ss.n_lists), dim3(64 * kF32Waves), head_dim == 64 ? f32_lds<64>() : f32_lds<128>(), st, p, ss);
            } else if (head_dim == 64) hipLaunchKernelGGL(hyd_bwd_dq_fp32_kernel<64>, grid_q, dim3(64 * kF32Waves), f32_lds<64>(), st, p);
            else if (short_rows) hipLaunchKernelGGL((hyd_bwd_dq_fp32_kernel<128, true>), grid_q, dim3(64 * kF32Waves), f32_rows_lds(), st, p);
            else hipLaunchKernelGGL(hyd_bwd_dq_fp32_kernel<128>, grid_q, dim3(64 * kF32Waves), f32_lds<128>(), st, p);
        }
        {
            p.hdr = sv_kv.hdr; p.items = sv_kv.exec; p.cursors = sv_kv.hdr + kHdrCursor; p.hm = head_map_kv(hkv, grid_kv.x);
            KernelTimer kt("bwd_dkdv_fp32", st);
            if (head_dim == 64) hipLaunchKernelGGL(hyd_bwd_dkdv_fp32_kernel<64>, grid_kv, dim3(64 * kF32KvWaves), f32_lds<64>(), st, p);
            else if (short_rows) hipLaunchKernelGGL((hyd_bwd_dkdv_fp32_kernel<128, true>), grid_kv, dim3(64 * kF32KvWaves), f32_rows_lds(), st, p);
            else hipLaunchKernelGGL(hyd_bwd_dkdv_fp32_kernel<128>, grid_kv, dim3(64 * kF32KvWaves), f32_lds<128>(), st, p);
        }
    }
    return hipGetLastError() == hipSuccess ? HYD_OK : HYD_ERR_LAUNCH;
}

}  // namespace

extern "C" {

hyd_status hyd_varlen_attn_fwd(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                               int num_seqs, const int32_t* cu_seqlens_host, int total_tokens,
                               int max_seqlen, int hq, int hkv, int head_dim, float softmax_scale,
                               hyd_dtype dt, void* o, float* lse, void* workspace,
                               size_t workspace_bytes, void* hip_stream) {
    return fwd_impl(q, k, v, cu_seqlens, num_seqs, cu_seqlens_host, nullptr, nullptr, false, total_tokens,
                    max_seqlen, hq, hkv, head_dim, softmax_scale, dt, o, lse, workspace, workspace_bytes,
                    hip_stream);
}

hyd_status hyd_varlen_attn_fwd_rope(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                                    int num_seqs, const int32_t* cu_seqlens_host, int total_tokens,
                                    int max_seqlen, int hq, int hkv, int head_dim, float softmax_scale,
                                    float rope_base, hyd_dtype dt, void* o, float* lse, void* workspace,
                                    size_t workspace_bytes, void* hip_stream) {
    if (!(rope_base > 1.f)) return HYD_ERR_SHAPE;
    return fwd_impl(q, k, v, cu_seqlens, num_seqs, cu_seqlens_host, nullptr, nullptr, false, total_tokens,
                    max_seqlen, hq, hkv, head_dim, softmax_scale, dt, o, lse, workspace, workspace_bytes,
                    hip_stream, rope_base);
}

hyd_status hyd_varlen_attn_bwd_rope(const void* q, const void* k, const void* v, const void* o, const float* lse,
                                    const void* d_o, const int32_t* cu_seqlens, int num_seqs,
                                    const int32_t* cu_seqlens_host, int total_tokens, int max_seqlen, int hq,
                                    int hkv, int head_dim, float softmax_scale, float rope_base, hyd_dtype dt,
                                    void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes,
                                    void* hip_stream) {
    if (!(rope_base > 1.f)) return HYD_ERR_SHAPE;
    return bwd_impl(q, k, v, o, lse, d_o, cu_seqlens, num_seqs, cu_seqlens_host, nullptr, nullptr, false,
                    total_tokens, max_seqlen, hq, hkv, head_dim, softmax_scale, dt, dq, dk, dv, workspace,
                    workspace_bytes, hip_stream, rope_base);
}

size_t hyd_varlen_attn_fwd_noalloc_max_workspace(void) { return kScratchBytes; }

hyd_status hyd_varlen_attn_fwd_noalloc(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                                       int num_seqs, const int32_t* cu_seqlens_host, int total_tokens,
                                       int max_seqlen, int hq, int hkv, int head_dim, float softmax_scale,
                                       hyd_dtype dt, void* o, float* lse, void* hip_stream) {
    // sizes first (no HIP call yet): the forward's workspace for these sizes must fit the array
    if (total_tokens < 0 || num_seqs < 0) return HYD_ERR_SHAPE;
    if (hq <= 0 || hkv <= 0 || hq % hkv != 0) return HYD_ERR_HEADS;
    if (dt != HYD_BF16 && dt != HYD_FP32) return HYD_ERR_DTYPE;
    if (!head_dim_ok(dt, head_dim)) return HYD_ERR_HEADDIM;
    // (if need be with 256-row tiles and without the second copy of the item records)
    const bool compact = fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, false).used > kScratchBytes;
    if (compact && fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, true).used > kScratchAll) return HYD_ERR_WORKSPACE;
    // the rest of the argument checks, still before any HIP call (a stand-in for the workspace pointer)
    const hyd_status vs = validate_common(cu_seqlens, num_seqs, cu_seqlens_host, total_tokens, max_seqlen, hq, hkv, head_dim,
                                          dt, reinterpret_cast<const void*>(kAlign), kScratchAll, false, compact, true);
    if (vs != HYD_OK) return vs;
    if (total_tokens == 0 || num_seqs == 0) return HYD_OK;
    if (!q || !k || !v || !o || !lse) return HYD_ERR_NULL;
    DeviceInfo* dev = nullptr;
    const hyd_status ds = device_info(&dev);          // first call on a device: looks the array's address up
    if (ds != HYD_OK) return ds;
    return fwd_impl(q, k, v, cu_seqlens, num_seqs, cu_seqlens_host, nullptr, nullptr, false, total_tokens, max_seqlen,
                    hq, hkv, head_dim, softmax_scale, dt, o, lse, dev->scratch, kScratchAll, hip_stream, 0.f, compact, true);
}

hyd_status hyd_varlen_attn_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse,
                               const void* d_o, const int32_t* cu_seqlens, int num_seqs,
                               const int32_t* cu_seqlens_host, int total_tokens, int max_seqlen, int hq,
                               int hkv, int head_dim, float softmax_scale, hyd_dtype dt, void* dq, void* dk,
                               void* dv, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return bwd_impl(q, k, v, o, lse, d_o, cu_seqlens, num_seqs, cu_seqlens_host, nullptr, nullptr, false,
                    total_tokens, max_seqlen, hq, hkv, head_dim, softmax_scale, dt, dq, dk, dv, workspace,
                    workspace_bytes, hip_stream);
}

hyd_status hyd_varlen_attn_fwd_range(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                                     int num_seqs, const int32_t* cu_seqlens_host, const int32_t* ranges,
                                     const int32_t* ranges_host, int total_tokens, int max_seqlen, int hq,
                                     int hkv, int head_dim, float softmax_scale, hyd_dtype dt, void* o,
                                     float* lse, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return fwd_impl(q, k, v, cu_seqlens, num_seqs, cu_seqlens_host, ranges, ranges_host, true, total_tokens,
                    max_seqlen, hq, hkv, head_dim, softmax_scale, dt, o, lse, workspace, workspace_bytes,
                    hip_stream);
}

hyd_status hyd_varlen_attn_bwd_range(const void* q, const void* k, const void* v, const void* o,
                                     const float* lse, const void* d_o, const int32_t* cu_seqlens,
                                     int num_seqs, const int32_t* cu_seqlens_host, const int32_t* ranges,
                                     const int32_t* ranges_host, int total_tokens, int max_seqlen, int hq,
                                     int hkv, int head_dim, float softmax_scale, hyd_dtype dt, void* dq,
                                     void* dk, void* dv, void* workspace, size_t workspace_bytes,
                                     void* hip_stream) {
    return bwd_impl(q, k, v, o, lse, d_o, cu_seqlens, num_seqs, cu_seqlens_host, ranges, ranges_host, true,
                    total_tokens, max_seqlen, hq, hkv, head_dim, softmax_scale, dt, dq, dk, dv, workspace,
                    workspace_bytes, hip_stream);
}

hyd_status hyd_attn_merge(const void* o_a, const float* lse_a, const void* o_b, const float* lse_b,
                          int total_tokens, int hq, int head_dim, hyd_dtype dt, void* o_out, float* lse_out,
                          void* hip_stream) {
    if (dt != HYD_BF16) return HYD_ERR_DTYPE;
    if (total_tokens < 0) return HYD_ERR_SHAPE;
    if (hq <= 0) return HYD_ERR_HEADS;
    if (!head_dim_ok(dt, head_dim)) return HYD_ERR_HEADDIM;
    if (total_tokens == 0) return HYD_OK;
    if (!o_a || !lse_a || !o_b || !lse_b || !o_out || !lse_out) return HYD_ERR_NULL;
    DeviceInfo* dev = nullptr;
    const hyd_status ds = device_info(&dev);
    if (ds != HYD_OK) return ds;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    {
        KernelTimer kt("merge_bf16", st);
        const int chunks = merge_chunks(hq);
        const bool apart = o_out != o_a && o_out != o_b;
        const bool brief = apart && head_dim == kHeadDim && hq >= kMergeHeads && 6ll * total_tokens * hq * head_dim > kMergeCached;
        const int most = brief ? kMergeShortTok : kMergeTok;
        int log2_tok = 0;
        while ((2 << log2_tok) <= most && ((long long)total_tokens >> (log2_tok + 1)) * chunks >= kMergeGroups) ++log2_tok;
        const dim3 mgrid((unsigned)(((long long)total_tokens + (1 << log2_tok) - 1) >> log2_tok) * (unsigned)chunks);
        const auto kernel = head_dim == 64 ? hyd_merge_bf16_kernel<64>
                                           : brief ? hyd_merge_bf16_kernel<kHeadDim, kMergeShortThreads, kMergeShortTok, 1> : hyd_merge_bf16_kernel<kHeadDim>;
        hipLaunchKernelGGL(kernel, mgrid, dim3(brief ? kMergeShortThreads : kMergeThreads), 0, st, static_cast<const uint16_t*>(o_a), lse_a,
                           static_cast<const uint16_t*>(o_b), lse_b, static_cast<uint16_t*>(o_out), lse_out, total_tokens, hq, chunks, log2_tok);
    }
    return hipGetLastError() == hipSuccess ? HYD_OK : HYD_ERR_LAUNCH;
}

hyd_status hyd_rope_packed(const void* x, const int32_t* cu_seqlens, int num_seqs, int total_tokens, int heads,
                           int head_dim, float base, int inverse, hyd_dtype dt, void* out, void* hip_stream) {
    if (dt != HYD_BF16) return HYD_ERR_DTYPE;
    if (total_tokens < 0 || num_seqs < 0 || (num_seqs == 0 && total_tokens != 0) || !(base > 1.f)) return HYD_ERR_SHAPE;
    if (heads <= 0) return HYD_ERR_HEADS;
    if (!head_dim_ok(dt, head_dim)) return HYD_ERR_HEADDIM;
    if (total_tokens == 0) return HYD_OK;
    if (!x || !cu_seqlens || !out) return HYD_ERR_NULL;
    DeviceInfo* dev = nullptr;
    const hyd_status ds = device_info(&dev);
    if (ds != HYD_OK) return ds;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    {
        KernelTimer kt("rope_bf16", st);
        const dim3 rgrid((unsigned)((total_tokens + kRopeTok - 1) / kRopeTok));
        if (head_dim == 64)
            hipLaunchKernelGGL(hyd_rope_bf16_kernel<64>, rgrid, dim3(kRopeThreads), 0, st, static_cast<const uint16_t*>(x), cu_seqlens,
                               num_seqs, total_tokens, heads, log2((double)base), inverse != 0, static_cast<uint16_t*>(out));
        else
            hipLaunchKernelGGL(hyd_rope_bf16_kernel<kHeadDim>, rgrid, dim3(kRopeThreads), 0, st, static_cast<const uint16_t*>(x), cu_seqlens,
                               num_seqs, total_tokens, heads, log2((double)base), inverse != 0, static_cast<uint16_t*>(out));
    }
    return hipGetLastError() == hipSuccess ? HYD_OK : HYD_ERR_LAUNCH;
}

hyd_status hyd_varlen_attn_schedule_layout(int total_tokens, int num_seqs, int hq, int hkv, int head_dim, hyd_dtype dt,
                                           int is_bwd, int which, size_t* header_offset, size_t* items_offset,
                                           int* max_items, int* tile) {
    if (!header_offset || !items_offset || !max_items || !tile) return HYD_ERR_NULL;
    if (total_tokens < 0 || num_seqs < 0 || which < 0 || which > 1 || (which == 1 && !is_bwd)) return HYD_ERR_SHAPE;
    if (hq <= 0 || hkv <= 0 || hq % hkv != 0) return HYD_ERR_HEADS;
    if (dt != HYD_BF16 && dt != HYD_FP32) return HYD_ERR_DTYPE;
    if (!head_dim_ok(dt, head_dim)) return HYD_ERR_HEADDIM;
    const WsLayout w = is_bwd ? bwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt)
                              : fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, false);
    const SchedLayout& v = w.sched[which];
    *header_offset = v.hdr; *items_offset = v.items; *max_items = v.max_items;
    *tile = is_bwd && which == 0 ? tile_kv(dt) : tile_q(dt);
    return HYD_OK;
}

hyd_status hyd_varlen_attn_schedule_status(const void* workspace, size_t workspace_bytes, int total_tokens, int num_seqs,
                                           int hq, int hkv, int head_dim, hyd_dtype dt, int is_bwd, void* hip_stream) {
    size_t hdr = 0, items = 0;
    int max_items = 0, tile = 0;
    const hyd_status ls = hyd_varlen_attn_schedule_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, is_bwd, 0, &hdr, &items,
                                                          &max_items, &tile);
    if (ls != HYD_OK) return ls;
    if (total_tokens == 0 || num_seqs == 0) return HYD_OK;
    const WsLayout w = is_bwd ? bwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt) : fwd_layout(total_tokens, num_seqs, hq, hkv, head_dim, dt, false);
    if (!workspace || workspace_bytes < w.need) return HYD_ERR_WORKSPACE;
    int head[2] = {0, 0};
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (hipMemcpyAsync(head, static_cast<const char*>(workspace) + hdr, sizeof(head), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return HYD_ERR_LAUNCH;
    if (head[kHdrFlags] & kSchedBadSeqlens) return HYD_ERR_SEQLENS;
    if (head[kHdrFlags] & kSchedTooLong) return HYD_ERR_SHAPE;
    return HYD_OK;
}

void hyd_enable_kernel_timing(int on) {
    t_timing = on != 0;
    timed_clear();
}

int hyd_kernel_times(const char** names, float* ms, int cap) {
    int n = 0;
    for (auto& t : t_timed) {
        if (n >= cap) break;
        float dt = 0.f;
        if (hipEventSynchronize(t.e1) != hipSuccess || hipEventElapsedTime(&dt, t.e0, t.e1) != hipSuccess) dt = -1.f;
        names[n] = t.name;
        ms[n] = dt;
        ++n;
    }
    timed_clear();
    return n;
}

void hyd_set_wg_trace(void* device_records, int capacity_records) {
    t_trace.rec = static_cast<unsigned long long*>(device_records);
    t_trace.capacity = device_records ? capacity_records : 0;
}

}  // extern "C"
