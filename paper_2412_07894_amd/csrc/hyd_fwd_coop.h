// bf16 forward for launches that last as long as their longest item: 64 query rows per workgroup, four waves to 32 of them.
// See hyd_fwd_bf16.h for the arithmetic, the orientation and the reference of a row.
//
// A step covers 128 keys.  Of the waves that share 32 rows, each forms the scores and the probabilities of one
// 32-key block, the probabilities meet in LDS, and each takes a quarter of the head dimension through all four blocks: every
// sum has the terms and the order it has in the other forms, whose results these are bit for bit (but for rows
// whose sum has passed kRefSlack between the two tiles of a step: O and l are scaled back behind the step).
// For 128 keys the longest item of a launch goes through one step of 32 products per SIMD where the half tiles of
// QuerySplit<1> go through two of 32 by a single wave each: 1.36 us against 1.84 (one sequence of 3000 tokens, 8 heads 52.4 -> 41.6
// us).  A step is bound by the two dependent products and their trips through LDS, which carries 256 KB of fragments,
// probabilities and tiles in it (2000 clocks of 2850); on a full chip the form takes 1.8 times what whole tiles take.
#pragma once
#include "hyd_fwd_bf16.h"

namespace hyd {

constexpr int kCoRows = 64, kCoGroups = 4, kCoKeys = 32 * kCoGroups;
constexpr int kCoStageBytes = 2 * kFwdStageBytes;                     // two 64-key tiles of K and V
constexpr int kCoQOff = 2 * kCoStageBytes;                            // the item's Q rows, then the probabilities of a step
constexpr int kCoMaxOff = kCoQOff + kCoRows * kRowBytes;              // [row block][group][32 rows][largest, smallest score]
constexpr int kCoSlotOff = kCoMaxOff + 2 * kCoGroups * 32 * 8;        // work slot (64 bytes), overflow and care flags
constexpr int kCoTabOff = kCoSlotOff + 128;                           // rotary frequencies (kSelf)
constexpr int kCoLds = kCoTabOff + kHeadDim / 2 * 8;

// (for a head dimension of 128: with 64, two of the four waves would have no part in the second product)
template <bool kSelf>
__device__ __forceinline__ void fwd_coop_items(const FwdParams& p, const SelfSchedule* ss, char* smem) {
    constexpr int D = kHeadDim, kRowB = D * 2, NK = D / 16, NDB = D / 32;
    static_assert(NDB == kCoGroups, "a quarter of the head dimension each");
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4_w;
    typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
    int* slot = reinterpret_cast<int*>(smem + kCoSlotOff);
    volatile int* redo = slot + 16;
    volatile int* care_flag = slot + 17;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave & 1, kg = wave >> 1;                          // row block, key block of a step and quarter of the head dimension
    const int l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const int64_t q_stride = (int64_t)p.hq * D, kv_stride = (int64_t)p.hkv * D;
    const uint32_t kv_stride_b = (uint32_t)kv_stride * 2, q_stride_b = (uint32_t)q_stride * 2;
    const unsigned long long t_start = p.tr.rec ? wall_clock64() : 0ull;
    unsigned long long n_done = 0;

    FragAddr fa;
    fa.init(lane, smem);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const uint32_t k_block = (uint32_t)((kg >> 1) * kFwdStageBytes + (kg & 1) * 32 * kRowBytes);      // this wave's keys in a stage
    uint32_t v_lo = fa.col[0], v_hi = fa.col[1];
#pragma unroll
    for (int i = 1; i < NDB; ++i)
        if (kg == i) { v_lo = fa.col[2 * i]; v_hi = fa.col[2 * i + 1]; }
    const uint32_t p_at = lds0 + (uint32_t)(kCoQOff + rb * 8 * 1024 + lane * 16);                    // probabilities: [row block][8 key steps][lane]
    const uint32_t max_at = lds0 + (uint32_t)(kCoMaxOff + (rb * kCoGroups * 32 + l32) * 8);          // [group]
    const int dma_row = 4 * wave + (lane >> 4);
    const uint32_t dma_voff = dma_lane_voff<D>(dma_row, lane, kv_stride_b);
    const uint32_t dma_voff_q = dma_lane_voff<D>(dma_row, lane, q_stride_b);
    const uint32_t tile_bytes = kFwdBN * kv_stride_b;
    const float scale_log2 = fmaxf(fabsf(p.scale_log2), 1e-30f);
    const uint32_t sign_flip = p.scale_log2 < 0.f ? 0x80008000u : 0u;

    WorkFetcher wf;
    WorkItem wi;
    bool have;
    if constexpr (kSelf) have = self_first(*ss, smem, kFwdThreads, wi);
    else have = wf.first(p.hm, p.hdr, p.cursors, p.items, slot, wi, blockIdx.x);
    const double* rope_tab = p.rope_tab;
    while (have) {
        ++n_done;
        const auto same = [](int x) { return __builtin_amdgcn_readfirstlane(x); };      // (the item is the workgroup's)
        const int head = same(wi.head), row0 = same(wi.row0), L = same(wi.len);
        const int td = same(wi.lev) - 1, q0 = td * kCoRows;           // diagonal (= last) tile; first row
        const int kv_end = min(L, q0 + kCoRows);
        const int n_kt = td + 1, n_steps = (n_kt + 1) / 2;
        const int g = head / G;
        const int wrow0 = q0 + 32 * rb, qrow = wrow0 + l32;
        const bool active = wrow0 < L;
        const uint32_t kv_bytes = (uint32_t)(kv_end - 1) * kv_stride_b + kRowB;
        const __amdgpu_buffer_rsrc_t rk = make_rsrc(p.k + (int64_t)row0 * kv_stride + (int64_t)g * D, kv_bytes);
        const __amdgpu_buffer_rsrc_t rv = make_rsrc(p.v + (int64_t)row0 * kv_stride + (int64_t)g * D, kv_bytes);
        auto dma_step = [&](int s, int stage) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int t = 2 * s + x;
                if (t >= n_kt) break;
                char* dst = smem + stage * kCoStageBytes + x * kFwdStageBytes + 4 * wave * kRowBytes;
#pragma unroll
                for (int j = 0; j < 16 / kFwdWaves; ++j) {
                    const uint32_t soff = (uint32_t)t * tile_bytes + (uint32_t)(j * kFwdWaves * 4) * kv_stride_b;
                    char* d = dst + j * kFwdWaves * 4 * kRowBytes;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void*)d, 16, dma_voff, soff, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(d + kFwdTileBytes), 16, dma_voff, soff, 0, 0);
                }
            }
        };
        {
            const uint32_t q_bytes = (uint32_t)(min(L - q0, kCoRows) - 1) * q_stride_b + kRowB;
            dma_rows<kFwdWaves>(make_rsrc(p.q + (int64_t)(row0 + q0) * q_stride + (int64_t)head * D, q_bytes), smem,
                                [](int) { return kCoQOff; }, 1, q_stride_b, [](int) { return 0u; }, wave, dma_voff_q);
        }
        dma_step(0, 0);
        if (tid == 0) { *redo = 0; *care_flag = 0; }
        if (kSelf && rope_tab) {
            double* tab = reinterpret_cast<double*>(smem + kCoTabOff);
            rope_table_fill(tab, D / 2, ss->log2_base, tid, kFwdThreads);
            rope_tab = tab;
        }
        __syncthreads();                                              // the first tiles and the Q rows have landed
        bf16x8 qf[NK];
        {
            u32x4 qv[NK];
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) qv[ks] = *(lds_u32x4*)(uintptr_t)(fa.row[ks] + (uint32_t)(kCoQOff + rb * 32 * kRowBytes));
            __builtin_amdgcn_s_waitcnt(0xc07f);                       // lgkmcnt(0)
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) asm volatile("" : "+v"(qv[ks]));       // the reads stay on this side of the barrier
            if (rope_tab) rope_row_frags<D, false>(qv, rope_tab, qrow, half);
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) qf[ks] = as_bf16x8(qv[ks] ^ sign_flip);
        }
        __builtin_amdgcn_s_barrier();                                 // probabilities may take the place of Q
        const bool short_item = n_steps <= kShortItem;
        if (!kSelf && short_item) wf.claim(p.hm, p.cursors);

        f32x16 acc;
        float m_ref, l_run;
        bool overflow = false, again = false;                         // again: the item is repeated with care
        while (true) {
            m_ref = -INFINITY;
            l_run = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            bool care = again;                                        // of this row block
            auto step = [&](auto stage_tag, int s) {
                constexpr int ST = decltype(stage_tag)::value, base = ST * kCoStageBytes;
                const bool search = s == 0 || same(*care_flag) != 0;  // (read while no load is under way: it would be waited for)
                if (s + 1 < n_steps) dma_step(s + 1, ST ^ 1);
                const int t = 2 * s + (kg >> 1);                      // this wave's tile
                const bool work = active && t <= td;
                f32x16 x;
                if (work) {
                    constexpr int kAhead = NK < 6 ? NK : 6;
                    bf16x8 kf[kAhead];
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[r] = 0.f;
#pragma unroll
                    for (int i = 0; i < kAhead; ++i) kf[i] = as_bf16x8(*(lds_u32x4*)(uintptr_t)(fa.row[i] + k_block + (uint32_t)base));
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < NK; ++i) {
                        x = mfma32(kf[i % kAhead], qf[i], x);
                        if (i + kAhead < NK) kf[i % kAhead] = as_bf16x8(*(lds_u32x4*)(uintptr_t)(fa.row[i + kAhead] + k_block + (uint32_t)base));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (t == td) {
                        const int k0 = t * kFwdBN + 32 * (kg & 1) + 4 * half - qrow;
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (8 * (r >> 2) + (r & 3) + k0 > 0) x[r] = -INFINITY;
                    }
                }
                float m_of[2] = {m_ref, m_ref}, alpha_of[2] = {1.f, 1.f};       // reference and factor of O and l, by tile
                bool grow[2] = {false, false};
                if (search) {
                    // the row maxima (and, first, minima) of the blocks meet in LDS
                    if (work) {
                        float mx = x[0], mn = x[0], lo, hi;
#pragma unroll
                        for (int r = 1; r < 16; ++r) { mx = fmaxf(mx, x[r]); mn = fminf(mn, x[r]); }
                        both_halves(mx, lo, hi);
                        mx = fmaxf(lo, hi);
                        both_halves(mn, lo, hi);
                        mn = fminf(lo, hi);
                        *(lds_f32x2*)(uintptr_t)(max_at + (uint32_t)(kg * 32 * 8)) = f32x2{mx, mn};
                    }
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    __builtin_amdgcn_s_barrier();
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        if (!active || 2 * s + y > td) continue;
                        const f32x2 a = *(lds_f32x2*)(uintptr_t)(max_at + (uint32_t)(2 * y * 32 * 8)), b = *(lds_f32x2*)(uintptr_t)(max_at + (uint32_t)((2 * y + 1) * 32 * 8));
                        const float cand = fmaxf(a[0], b[0]) * scale_log2;
                        if (s == 0 && y == 0) {
                            m_ref = cand;
                            if (__any(cand - fminf(a[1], b[1]) * scale_log2 > kRefSpread)) { care = true; *care_flag = 1; }
                        } else if (care && __any(cand > m_ref + kRefStep)) {
                            const float m_new = fmaxf(m_ref, cand);
                            alpha_of[y] = __builtin_amdgcn_exp2f(m_ref - m_new);
                            grow[y] = true;
                            m_ref = m_new;
                        }
                        m_of[y] = m_ref;
                        if (y == 0) m_of[1] = m_ref;
                    }
                }
                if (work) {
                    const float m = m_of[kg >> 1];
                    u32x4 pk[2];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * j], scale_log2, -m));
                        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * j + 1], scale_log2, -m));
                        pk[j >> 2][j & 3] = pack_bf16(p0, p1);
                    }
                    *(lds_u32x4_w*)(uintptr_t)(p_at + (uint32_t)(2 * kg * 1024)) = pk[0];
                    *(lds_u32x4_w*)(uintptr_t)(p_at + (uint32_t)((2 * kg + 1) * 1024)) = pk[1];
                }
                __builtin_amdgcn_s_waitcnt(0xc07f);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (active) {
                    constexpr int kAhead = 3;
                    LdsQueue lq{0};
                    RowFrag pf[kAhead];
                    ColFrag vf[kAhead];
                    auto issue = [&](int b) {                         // key step b of the 8
                        lds_issue_row(lq, pf[b % kAhead], p_at, b * 1024);
                        constexpr int v = base + kFwdTileBytes;
                        const int off = v + (b >> 2) * kFwdStageBytes + (b & 3) * 16 * kRowBytes, hi = off & ~0xffff;
                        lds_issue_col(lq, vf[b % kAhead], v_lo + (uint32_t)hi, v_hi + (uint32_t)hi, off - hi);
                    };
#pragma unroll
                    for (int y = 0; y < 2; ++y) {
                        if (2 * s + y > td) break;
                        if (grow[y]) {
                            l_run *= alpha_of[y];
#pragma unroll
                            for (int r = 0; r < 16; ++r) acc[r] *= alpha_of[y];
                        }
                        float lsum = 0.f;
#pragma unroll
                        for (int b = 0; b < kAhead; ++b) issue(4 * y + b);
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const int n = 4 * y + b;
                            const bf16x8 pb = lds_wait(lq, pf[n % kAhead]);
                            const bf16x8 v = lds_wait(lq, vf[n % kAhead]);
                            acc = mfma32(v, pb, acc);
                            u32x4 w;
                            __builtin_memcpy(&w, &pb, 16);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {             // row sum of the ROUNDED probabilities
                                bf16x2 pr;
                                const uint32_t u = w[e];
                                __builtin_memcpy(&pr, &u, 4);
                                const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
                                lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, lsum, false);
                            }
                            if (b + kAhead < 4) issue(n + kAhead);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        l_run += lsum;
                    }
                    if (__builtin_expect(__any(l_run > kRefSlack), 0)) {
                        float lo, hi;
                        both_halves(l_run, lo, hi);
                        const uint32_t e = __float_as_uint(fmaxf(lo, hi)) >> 23;
                        const f32x16 one[1] = {acc};
                        const uint32_t big = max(e << 23, largest_bits(one));
                        const int k = e > 127u ? min((int)e - 127, 126) : 0;
                        const float m_new = m_ref + (float)k, moved = m_new - m_ref;
                        // (whether O is finite may differ between the waves of a row; the item is repeated then)
                        const bool ok = (e << 23) < kInfBits && moved <= 126.f;
                        const float alpha = ok ? __builtin_amdgcn_exp2f(-moved) : 1.f;
                        if (!ok || big >= kInfBits) overflow = true;
                        l_run *= alpha;
                        m_ref = ok ? m_new : m_ref;
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] *= alpha;
                    }
                }
                __builtin_amdgcn_s_waitcnt(0x0070);                   // vmcnt(0), lgkmcnt(0)
                __builtin_amdgcn_s_barrier();
            };
            for (int s = 0; s < n_steps; s += 2) {
                step(std::integral_constant<int, 0>{}, s);
                if (s + 1 < n_steps) step(std::integral_constant<int, 1>{}, s + 1);
            }
            if (__any(l_run > kRefQuiet)) {
                const f32x16 one[1] = {acc};
                overflow |= largest_bits(one) >= kInfBits;
            }
            if (!care && __any(overflow)) *redo = 1;
            __syncthreads();
            if (__builtin_expect(*redo == 0, 1)) break;
            again = true;
            __syncthreads();
            if (tid == 0) { *redo = 0; *care_flag = 1; }
            dma_step(0, 0);
            __syncthreads();
        }
        if (!kSelf && !short_item) wf.claim(p.hm, p.cursors);
        float l_lo, l_hi;
        both_halves(l_run, l_lo, l_hi);
        const float l_tot = l_lo + l_hi, inv = 1.f / l_tot;
        // O: the quarters of a row meet in 8 KB of the ring per row block and leave as whole rows, 8 rows per wave
        {
            const uint32_t o_stage = lds0 + (uint32_t)(rb * 32 * kRowBytes);
            if (active) {
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    const u32x2 w = {pack_bf16(acc[4 * rq] * inv, acc[4 * rq + 1] * inv), pack_bf16(acc[4 * rq + 2] * inv, acc[4 * rq + 3] * inv)};
                    *(lds_u32x2*)(uintptr_t)(o_stage + (uint32_t)(l32 * kRowBytes + 8 * half + (((4 * kg + rq) ^ swz(l32)) << 4))) = w;
                }
            }
            __syncthreads();
            if (active) {
                const int c16 = lane & 15;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = 8 * kg + 4 * i + (lane >> 4);
                    const u32x4 w = *(lds_u32x4*)(uintptr_t)(o_stage + (uint32_t)(r * kRowBytes + ((c16 ^ swz(r)) << 4)));
                    if (wrow0 + r < L)
                        *reinterpret_cast<u32x4*>(p.o + (int64_t)(row0 + wrow0 + r) * q_stride + (int64_t)head * D + 8 * c16) = w;
                }
                if (kg == 0 && half == 0 && qrow < L)
                    p.lse[(int64_t)head * p.T + row0 + qrow] = (m_ref + __builtin_amdgcn_logf(l_tot)) * 0.69314718055994530942f;
            }
        }
        if constexpr (kSelf) have = false;
        else have = wf.next(p.hm, p.cursors, p.items, slot, wi);
    }
    trace_write(p.tr, 0, t_start, n_done);
}

__global__ void __launch_bounds__(kFwdThreads, 1) hyd_fwd_coop_bf16_kernel(FwdParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    fwd_coop_items<false>(p, nullptr, smem);
}
__global__ void __launch_bounds__(kFwdThreads, 1) hyd_fwd_coop_self_bf16_kernel(FwdParams p, SelfSchedule ss) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    fwd_coop_items<true>(p, &ss, smem);
}

}  // namespace hyd
