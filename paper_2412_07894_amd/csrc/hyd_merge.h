// Merge of two partial attention results over the same rows (context parallelism: each partial
// comes from one chunk of the keys, arXiv 2412.07894 Sec. 2.1).  With LSE_x = ln sum exp(s) over
// the keys of partial x, the softmax over the union of the keys is
//     LSE = ln(exp(LSE_a) + exp(LSE_b)),   O = exp(LSE_a - LSE) O_a + exp(LSE_b - LSE) O_b;
// a partial that saw no key carries LSE = -inf and O = 0 and is the neutral element.
//
// Bound by HBM, so rows that need no work are not touched: a visit of a context-parallel ring merges buffers
// of all T rows of which only the rank's own carry a partial, and where LSE_b = -inf (or LSE_a) a merge in place
// leaves the other partial's row as it is.  A workgroup takes 32 tokens of up to 8 heads: the weights of its rows are
// formed first, a thread per row, so that the [Hq][T] vectors are read and written in runs of 32
// floats; then kLanes lanes per row move 16 bytes each, four rows in flight.  Measured (16384 tokens, 32 heads): a merge
// in place of 3030 tokens' rows 64 us before (event times), 27 now.
//   Few rows: workgroups of fewer tokens, as long as there are 1024 of them, since one of 32 tokens loops over its rows
// while CUs idle (one-row workgroups of 16 lanes before, 32 tokens always, now: 64 tokens, 8 heads 7.5, 9.4, 7.2 us; 2369 7.5, 10.4, 7.3;
// 4000 tokens, 16 heads 8.3, 13.1, 7.4; 2369, 32 heads 10.4, 16.9, 9.1).
//   Many rows that all move: the order of the accesses counts, which is that of the memory where workgroups are short and keep one
// row per lane in flight.  A merge out of place, which moves every row, of more than the caches hold takes workgroups of 4 tokens
// and 512 threads (d = 128: 16384 tokens, 32 heads 71, 82, 72 us; 33000 141, 164, 140; 131072, 8 heads 138, 157, 140; 10 heads 176, 196,
// 186).  In place the long workgroups stay: they pass over rows without a partial in half the time (33000 tokens, 32 heads, a quarter of the
// rows 141, 39, short ones 69), which costs a merge in place of all rows a sixth (141, 166, short ones 140).
#pragma once
#include "hyd_device.h"

namespace hyd {

constexpr int kMergeThreads = 256, kMergeTok = 32, kMergeHeads = 8, kMergeGroups = 1024;
constexpr int kMergeShortThreads = 512, kMergeShortTok = 4;
constexpr long long kMergeCached = 300ll << 20;            // bytes of O, of three buffers
inline int merge_chunks(int hq) { return (hq + kMergeHeads - 1) / kMergeHeads; }      // of the heads

// o_out / lse_out may alias either input (what is overwritten has been read before).
template <int D = kHeadDim, int kThreads = kMergeThreads, int kTok = kMergeTok, int kU = 4>          // kU: rows of a lane in flight
__global__ void __launch_bounds__(kThreads) hyd_merge_bf16_kernel(const uint16_t* o_a, const float* lse_a,
                                                                  const uint16_t* o_b, const float* lse_b,
                                                                  uint16_t* o_out, float* lse_out, int T, int hq, int chunks, int log2_tok) {
    __shared__ float wt[2][kTok * kMergeHeads];
    const int tid = threadIdx.x, per = (hq + chunks - 1) / chunks;             // heads of a chunk
    const int t0 = (int)(blockIdx.x / (unsigned)chunks) << log2_tok, h0 = (int)(blockIdx.x % (unsigned)chunks) * per;
    const int nt = min(1 << log2_tok, T - t0), nh = min(per, hq - h0);
    if (nh <= 0) return;
    {
        const int tl = tid & ((1 << log2_tok) - 1), hl = tid >> log2_tok;
        if (tl < nt && hl < nh) {
            const int64_t si = (int64_t)(h0 + hl) * T + t0 + tl;
            const float la = lse_a[si], lb = lse_b[si];
            const float m = fmaxf(la, lb);
            float ca = 0.f, cb = 0.f, lse = -INFINITY;
            if (m > -INFINITY) {
                constexpr float kL2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;
                const float wa = __builtin_amdgcn_exp2f((la - m) * kL2e), wb = __builtin_amdgcn_exp2f((lb - m) * kL2e);
                const float tot = wa + wb;                        // in [1, 2]
                lse = m + __builtin_amdgcn_logf(tot) * kLn2;
                const float inv = 1.f / tot;
                ca = wa * inv; cb = wb * inv;
            }
            wt[0][tl * per + hl] = ca;
            wt[1][tl * per + hl] = cb;
            lse_out[si] = lse;
        }
    }
    __syncthreads();
    constexpr int kLanes = D / 8, kGrps = kThreads / kLanes;                   // lanes per row, rows at a time
    const int c = tid % kLanes, n_rows = nt * per;
    const bool in_a = o_out == o_a, in_b = o_out == o_b;
    for (int r0 = tid / kLanes; r0 < n_rows; r0 += kGrps * kU) {
        u32x4 a[kU], b[kU];
        float ca[kU], cb[kU];
        int64_t at[kU];
        bool on[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int r = r0 + kGrps * u, tl = r / per, hl = r - tl * per;
            on[u] = r < n_rows && hl < nh;
            ca[u] = cb[u] = 0.f;
            if (on[u]) { ca[u] = wt[0][r]; cb[u] = wt[1][r]; }
            // the whole weight on the row that is there already
            if ((in_a && ca[u] == 1.f && cb[u] == 0.f) || (in_b && cb[u] == 1.f && ca[u] == 0.f)) on[u] = false;
            at[u] = ((int64_t)(t0 + tl) * hq + h0 + hl) * D + c * 8;
            a[u] = b[u] = u32x4{0u, 0u, 0u, 0u};
            // a weight of zero must also silence a partial whose unwritten rows hold non-finite bits: it is not read
            if (on[u] && ca[u] != 0.f) a[u] = *reinterpret_cast<const u32x4*>(o_a + at[u]);
            if (on[u] && cb[u] != 0.f) b[u] = *reinterpret_cast<const u32x4*>(o_b + at[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            u32x4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                r[e] = pack_bf16(ca[u] * bf16_lo(a[u][e]) + cb[u] * bf16_lo(b[u][e]), ca[u] * bf16_hi(a[u][e]) + cb[u] * bf16_hi(b[u][e]));
            if (on[u]) *reinterpret_cast<u32x4*>(o_out + at[u]) = r;
        }
    }
}

}  // namespace hyd
