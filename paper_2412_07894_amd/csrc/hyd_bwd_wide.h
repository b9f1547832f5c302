// bf16 dK/dV, wide form: 256 keys per workgroup, 64 per wave.  See hyd_bwd_bf16.h for the arithmetic, the fragment
// convention and the narrow form (128 keys, a pair of waves for 32 of them), whose results this one gives bit for bit.
#pragma once
#include "hyd_bwd_bf16.h"

namespace hyd {

// Work item = (sequence, 256-key tile, KV head); 4 waves, one per SIMD, each of which owns 64 keys and takes
// all four products of its blocks of 32 query rows and 64 keys in its own registers: the 256 of dK^T and
// dV^T in the accumulation file, K and V fragments, S and dP in the other.
//
// Against the narrow form a fragment of Q or dO serves two products instead of one (half the LDS reads), the stream
// of Q and dO is read once for 256 keys instead of twice, P does not travel between waves, and there is one barrier for 64
// rows instead of two.  What two waves of a SIMD give there, vector work of one under the products of
// the other, has to come from the order of instructions here: see `block`.  No unit is saturated: matrix pipe busy 61 % of a CU's
// clocks, vector ALU 34 %, LDS 20 % (131072 tokens of heavy-tailed lengths, 40 heads).  Each direct-to-LDS load of a step stands in a
// loop over the lanes' descriptors, which the compiler does not know to be alike; with one wave for a SIMD nothing covers it.  131072 tokens,
// 64/8 heads, long sequences, narrow -> wide 38.0 -> 33.1 ms; d = 64, 32768 tokens of heavy-tailed lengths, 32 heads 2.06 -> 1.72 ms.  On the way there: products left to the
// compiler 352 registers in scratch; one loop with a choice of bodies 371; exponentials right behind their scores 34.9
// ms; pinned by empty assembly statements (a wait state each) 34.2; vector work in assembly 33.3.
//
// It pays where items are long, since a wave has its SIMD to itself while the rows of an item arrive and its results
// leave, and where there are many, since they are twice as large; the rule is in the host code.
constexpr int kKwWaves = 4, kKwBN = 64 * kKwWaves, kKwBM = 64, kKwThreads = 64 * kKwWaves, kKwStages = 4;
constexpr int kKwTileBytes = kKwBM * kRowBytes;                       // 16 KB
constexpr int kKwStageBytes = 2 * kKwTileBytes;                       // Q, dO
// While an item begins, ring stage 0 takes its first tile, stages 1 and 2 its K rows and the rest its V rows; the
// statistics of the stages and the work slot, behind the ring, share the bytes of the latter.
constexpr int kKwStatOff = kKwStages * kKwStageBytes;                 // [stage][LSE2, D][64]
constexpr int kKwSlotOff = kKwStatOff + kKwStages * 2 * kKwBM * 4;
constexpr int kKwVOff = 3 * kKwStageBytes;                            // V rows while an item begins
constexpr int kKwLds = kKwVOff + kKwBN * kRowBytes;                   // 160 KB: all of a CU's LDS
static_assert(kKwSlotOff + 64 <= kKwLds, "statistics and work slot lie behind the ring");

// The products in assembly, so that each accumulator is in the file it belongs in (left to the compiler, S and dP go
// through the accumulation file too, two more vector instructions per score and more registers than there are).
// The compiler does not know these as matrix instructions: what reads their results keeps the distance by hand.
__device__ __forceinline__ void mfma_zero(f32x16& d, bf16x8 a, bf16x8 b) {            // d = a b
    asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_from(f32x16& d, bf16x8 a, bf16x8 b, const f32x16& c) {      // d = a b + c
    asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "v"(b), "v"(c));
}
__device__ __forceinline__ void mfma_add(f32x16& d, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_acc(f32x16& d, bf16x8 a, u32x4 b) {             // b: just formed by vector instructions
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}

// The vector work between them, in assembly too: volatile statements keep their order.
__device__ __forceinline__ void v_scale(float& d, float s, float scale, uint32_t l) {            // d = s * scale + l
    asm volatile("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(s), "s"(scale), "v"(l));
}
__device__ __forceinline__ void v_exp2(float& a, float& b) {
    asm volatile("v_exp_f32 %0, %0\n\tv_exp_f32 %1, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void v_pack_f16(uint32_t& d, float a, float b) {                     // round to nearest even, as pack_f16
    asm volatile("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void v_mul_f16_f32(float& a, float& b, uint32_t h, float x, float y) {      // the halves of h times x and y
    asm volatile("v_fma_mix_f32 %0, %2, %3, 0 op_sel_hi:[1,0,0]\n\tv_fma_mix_f32 %1, %2, %4, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
                 : "=&v"(a), "=v"(b) : "v"(h), "v"(x), "v"(y));
}
// The fragment as it is, waited for as in lds_wait.
__device__ __forceinline__ u32x4 lds_wait_raw(const LdsQueue& q, RowFrag& f) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(f.v) : "i"(q.issued - f.seq < 15 ? q.issued - f.seq : 15));
    return f.v;
}

// The accumulators, in their file.
template <int N>
__device__ __forceinline__ void keep_acc(f32x16 (&a)[2][N], f32x16 (&b)[2][N]) {
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) asm volatile("" : "+a"(a[i / N][i % N]), "+a"(b[i / N][i % N]));
}

template <int D = kHeadDim>
__global__ void __launch_bounds__(kKwThreads, 1) hyd_bwd_dkdv_wide_bf16_kernel(BwdParams p, WorkList list) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    static_assert(D == 128 || D == 64, "head dimension");
    constexpr int kRowB = D * 2, NK = D / 16, NDB = D / 32;
    int* slot = reinterpret_cast<int*>(smem + kKwSlotOff);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const int64_t q_stride = (int64_t)p.hq * D, kv_stride = (int64_t)p.hkv * D;
    const uint32_t q_stride_b = (uint32_t)q_stride * 2, kv_stride_b = (uint32_t)kv_stride * 2;
    const unsigned long long t_start = p.tr.rec ? wall_clock64() : 0ull;
    unsigned long long n_done = 0;

    // Fragment addresses (see FragAddr): those of the contraction steps of a row fragment differ in bits 5-7 only, those of the
    // column blocks of a column fragment in bits 6-7 and its second row group in bit 5 besides 8 rows, so all follow from
    // two by exclusive or (with all sixteen kept through the tile loop there are not enough registers).
    uint32_t row_frag, col_frag;
    {
        FragAddr fa;
        fa.init(lane, smem);
        row_frag = fa.row[0];
        col_frag = fa.col[0];
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const int dma_row = 4 * wave + (lane >> 4);
    const uint32_t dma_voff = dma_lane_voff<D>(dma_row, lane, q_stride_b);
    const uint32_t dma_voff_kv = dma_lane_voff<D>(dma_row, lane, kv_stride_b);
    const uint32_t tile_bytes = kKwBM * q_stride_b;
    const float scale_log2 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(fmaxf(fabsf(p.scale_log2), 1e-30f))));
    const uint32_t sign_flip = p.scale_log2 < 0.f ? 0x80008000u : 0u;
    PartialMaxima pm;
    pm.load(p.sc, lane);

    WorkFetcher wf;
    WorkItem wi;
    bool have = wf.first(list.hm, list.hdr, list.cursors, list.items, slot, wi, blockIdx.x);
    const float unscale = pow2i(-pm.shift());                         // 2^-kg
    while (have) {
        __syncthreads();                                      // everybody has read the work slot: its bytes may be overwritten
        const int lev = wi.lev, g = wi.head, row0 = wi.row0, L = wi.len;
        const int n_tiles = (L + kKwBN - 1) / kKwBN;
        const int j0 = (n_tiles - lev) * kKwBN;
        n_done += (min(L - j0, kKwBN) + kKvBN - 1) / kKvBN;   // (the trace counts tiles of the list of whole tiles)
        const int wkey0 = j0 + 64 * wave;                     // first key of this wave
        const bool active = wkey0 < L;
        const int td = wkey0 / kKwBM;                         // query tile that holds the wave's diagonal
        const int qt_first = j0 / kKwBM;
        const int n_qt = (L + kKwBM - 1) / kKwBM - qt_first;
        const int n_iter = n_qt * G;
        const uint32_t q_bytes = (uint32_t)(L - 1) * q_stride_b + kRowB;
        const uint32_t stat_bytes = (uint32_t)L * 4;

        constexpr int kDmaPerStage = 2 * (16 / kKwWaves) + 1;
        int ld_qt = qt_first, ld_h = 0;
        // the tiles of iteration (ld_qt, ld_h); `stats`: with their statistics (not for the item's first tile)
        auto dma_stage = [&](int stage, bool stats) {
            const int h = g * G + ld_h, qt = ld_qt;
            if (++ld_h == G) { ld_h = 0; ++ld_qt; }
            const int64_t base = (int64_t)row0 * q_stride + (int64_t)h * D;
            const __amdgpu_buffer_rsrc_t rq = make_rsrc(p.sc.q16 + base, q_bytes);
            const __amdgpu_buffer_rsrc_t rdo = make_rsrc(p.sc.do16 + base, q_bytes);
            char* dst = smem + stage * kKwStageBytes + 4 * wave * kRowBytes;
#pragma unroll
            for (int j = 0; j < 16 / kKwWaves; ++j) {
                const uint32_t soff = (uint32_t)qt * tile_bytes + (uint32_t)(j * kKwWaves * 4) * q_stride_b;
                char* d = dst + j * kKwWaves * 4 * kRowBytes;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rq, (lds_void_b*)d, 16, dma_voff, soff, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rdo, (lds_void_b*)(d + kKwTileBytes), 16, dma_voff, soff, 0, 0);
            }
            if (stats) {
                const int which = wave == 0 ? 0 : 1;
                const float* src = (which == 0 ? p.sc.lse2 : p.sc.Dkv) + (int64_t)h * p.T + row0;
                const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, stat_bytes);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_b*)(smem + kKwStatOff + stage * 2 * kKwBM * 4 + which * kKwBM * 4),
                                                         4, (uint32_t)lane * 4, (uint32_t)qt * kKwBM * 4, 0, 0);
            }
        };
        const bool short_item = n_iter <= kShortItem;
        if (short_item) wf.claim(list.hm, list.cursors);
        float first_stat = 0.f;                               // waves 0 and 1: LSE2 and D of the first tile
        {
            const int r = qt_first * kKwBM + lane;
            if (wave < 2 && r < L) first_stat = (wave == 0 ? p.sc.lse2 : p.sc.Dkv)[(int64_t)(g * G) * p.T + row0 + r];
            dma_stage(0, false);
        }
        {
            const uint32_t k_bytes = (uint32_t)(min(L - j0, kKwBN) - 1) * kv_stride_b + kRowB;
            const int64_t off = (int64_t)(row0 + j0) * kv_stride + (int64_t)g * D;
            auto tile_at = [&](int j) { return (uint32_t)(64 * j) * kv_stride_b; };
            dma_rows<kKwWaves>(make_rsrc(p.sc.k16 + off, k_bytes), smem + kKwStageBytes, [](int j) { return j * kKwTileBytes; },
                               kKwBN / 64, kv_stride_b, tile_at, wave, dma_voff_kv);
            dma_rows<kKwWaves>(make_rsrc(p.v + off, k_bytes), smem + kKwVOff, [](int j) { return j * kKwTileBytes; },
                               kKwBN / 64, kv_stride_b, tile_at, wave, dma_voff_kv);
        }
        f32x16 dv[2][NDB], dk[2][NDB];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) dv[kb][db][r] = dk[kb][db][r] = 0.f;
        __syncthreads();                                      // tile 0 and the K / V rows have landed
        bf16x8 kf[2][NK], vf[2][NK];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            u32x4 a[NK], b[NK];
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                a[ks] = *(lds_u32x4*)(uintptr_t)((row_frag ^ (uint32_t)(ks << 5)) + (uint32_t)(kKwStageBytes + (64 * wave + 32 * kb) * kRowBytes));
                b[ks] = *(lds_u32x4*)(uintptr_t)((row_frag ^ (uint32_t)(ks << 5)) + (uint32_t)(kKwVOff + (64 * wave + 32 * kb) * kRowBytes));
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);               // lgkmcnt(0)
#pragma unroll
            for (int ks = 0; ks < NK; ++ks) {
                asm volatile("" : "+v"(a[ks]), "+v"(b[ks]));  // the reads stay on this side of the barrier
                kf[kb][ks] = as_bf16x8(a[ks] ^ sign_flip);
#pragma unroll
                for (int e = 0; e < 4; ++e) b[ks][e] = bf16x2_to_f16x2(b[ks][e]);
                vf[kb][ks] = as_bf16x8(b[ks]);
            }
        }
        __builtin_amdgcn_s_barrier();                         // stages 1 to 3 and the statistics may be written now
        if (wave < 2) *reinterpret_cast<float*>(smem + kKwStatOff + wave * kKwBM * 4 + lane * 4) = first_stat;
        if (n_iter > 1) dma_stage(1, true);
        if (n_iter > 2) dma_stage(2, true);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();

        uint32_t fa_row = row_frag, fa_col[2 * NDB];          // in the current stage
#pragma unroll
        for (int i = 0; i < 2 * NDB; ++i) fa_col[i] = (col_frag ^ (uint32_t)((i >> 1) << 6 | (i & 1) << 5)) + (i & 1 ? 8 * kRowBytes : 0);
        uint32_t stat = lds0 + kKwStatOff;
        // One block of 32 rows (rows 32*ib.. of the stage that fa points at) and the wave's 64 keys, or (kN = 1) its
        // first 32.  kMask: the last 32 of them are the diagonal block.
        //
        // The block is a row of slots, a product each: S, dP, dV, dK.  What vector work there is goes into the shadows of
        // the products, a few instructions each, in an order in which none waits for its predecessor: scores are
        // scaled in one slot, their exponentials taken in the next and rounded in a third; dS likewise in two.  P of the block's
        // second 16 rows and dS are formed under the second products, which need the first 16 rows first.
        // Fragments are read kAhead ahead; the first ones of the next block, at `next_row`, under dK's products.
        constexpr int kAhead = 4;
        RowFrag rf[kAhead];
        auto block = [&](auto n_tag, auto mask_tag, int ib, uint32_t next_row) {
            constexpr int kN = decltype(n_tag)::value;        // key blocks
            constexpr bool kMask = decltype(mask_tag)::value;
            constexpr int kDp = NK * kN, kDv = 2 * kDp;               // first slots of dP and dV
            constexpr int kPairs = 8 * kN;                    // pairs of scores a lane holds; m = kN * j + kb is pair j of key block kb
            // pairs whose exponentials are begun by slot e behind kDp, whose dS by slot e behind kDsFrom
            constexpr int kExpNum = kN == 1 ? 128 / D : (D == 128 ? 2 : 3), kExpDen = kN == 1 ? 1 : (D == 128 ? 3 : 2);
            constexpr int kDsNum = 128 / D, kDsFrom = kN == 2 && D == 128 ? 40 : (kN == 2 || D == 128 ? 19 : 9);
            auto exp_count = [](int e) { const int n = e < 0 ? 0 : ((e + 1) * kExpNum + kExpDen - 1) / kExpDen; return n < kPairs ? n : kPairs; };
            auto ds_count = [](int e) { const int n = e < 0 ? 0 : (e + 1) * kDsNum; return n < kPairs ? n : kPairs; };
            LdsQueue lq{0};
            RowFrag l4[4], d4[4];
            ColFrag cf[kAhead];
            f32x16 s[kN], x[kN];
            uint32_t pk[kN][8], ds[kN][8];
            float arg[kPairs][2];
            const uint32_t sa = stat + (uint32_t)(32 * ib + 4 * half) * 4;
            // fragment i of the first products: Q rows, contraction step i (i < NK), then dO rows
            auto issue_first = [&](int i) {
                lds_issue_row(lq, rf[i % kAhead], fa_row ^ (uint32_t)((i % NK) << 5), (i < NK ? 0 : kKwTileBytes) + ib * 32 * kRowBytes);
            };
            // fragment i of the second products: dO columns, (contraction step, column block) = (i / NDB, i % NDB), then Q columns
            auto issue_second = [&](int i) {
                const int j = i % (2 * NDB);
                lds_issue_col(lq, cf[i % kAhead], fa_col[2 * (j % NDB)], fa_col[2 * (j % NDB) + 1],
                              (i < 2 * NDB ? kKwTileBytes : 0) + (2 * ib + j / NDB) * 16 * kRowBytes);
            };
            // the vector work of slot t
            auto shadow = [&](int t) {
                const int e = t - kDp, d = t - kDsFrom;
#pragma unroll
                for (int m = 0; m < kPairs; ++m)
                    if (m >= exp_count(e - 2) && m < exp_count(e - 1)) v_exp2(arg[m][0], arg[m][1]);
#pragma unroll
                for (int m = 0; m < kPairs; ++m) {
                    const int kb = m % kN, j = m / kN, r = 2 * j;
                    if (m >= exp_count(e - 1) && m < exp_count(e)) {
                        if ((r & 3) == 0 && kb == 0) lds_wait_raw(lq, l4[r >> 2]);
                        v_scale(arg[m][0], s[kb][r], scale_log2, l4[r >> 2].v[r & 3]);
                        v_scale(arg[m][1], s[kb][r + 1], scale_log2, l4[r >> 2].v[(r & 3) + 1]);
                    }
                    if (m >= ds_count(d - 1) && m < ds_count(d)) v_mul_f16_f32(arg[m][0], arg[m][1], pk[kb][j], x[kb][2 * j], x[kb][2 * j + 1]);
                }
#pragma unroll
                for (int m = 0; m < kPairs; ++m) {
                    if (m >= exp_count(e - 3) && m < exp_count(e - 2)) v_pack_f16(pk[m % kN][m / kN], arg[m][0], arg[m][1]);
                    if (m >= ds_count(d - 2) && m < ds_count(d - 1)) v_pack_f16(ds[m % kN][m / kN], arg[m][0], arg[m][1]);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
#pragma unroll
            for (int i = 0; i < NK; ++i) {                    // S
                const bf16x8 f = lds_wait(lq, rf[i % kAhead]);
#pragma unroll
                for (int kb = 0; kb < kN; ++kb) {
                    if (i == 0) mfma_zero(s[kb], f, kf[kb][i]);
                    else mfma_add(s[kb], f, kf[kb][i]);
                }
                issue_first(i + kAhead);
                // the statistics, early enough to be there for the first product of dP
                constexpr int kPer = 8 / NK;                  // per step: -D at the block's rows in steps 0 .. 3 / kPer, then -LSE2
#pragma unroll
                for (int e = 0; e < kPer; ++e) {
                    const int n = kPer * i + e - kPer;
                    if (n >= 0 && n < 4) lds_issue_row(lq, d4[n], sa, kKwBM * 4 + 32 * n);
                    if (n == 4) lds_issue_row(lq, l4[0], sa, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (kMask) {
                asm volatile("s_nop 15" ::: "memory");        // the scores are there
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (l32 > 8 * (r >> 2) + 4 * half + (r & 3)) s[kN - 1][r] = -INFINITY;
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {                  // dP begins at -D
                const u32x4 v = lds_wait_raw(lq, d4[rq]);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[0][4 * rq + e] = __uint_as_float(v[e]);
            }
#pragma unroll
            for (int i = 0; i < NK; ++i) {                    // dP
                const bf16x8 f = lds_wait(lq, rf[i % kAhead]);
#pragma unroll
                for (int n = 0; n < kN; ++n) {
                    const int kb = i == 0 ? kN - 1 - n : n;   // x[0] holds -D: the other block takes it from there
                    if (i == 0 && kb == 1) mfma_from(x[kN - 1], f, vf[kN - 1][0], x[0]);
                    else mfma_add(x[kb], f, vf[kb][i]);
                    if (i == 0 && kN == 1) asm volatile("s_nop 11");          // the scores are there
                    // -LSE2 of the next rows (with all of it requested at once there are not enough registers)
                    constexpr int kEvery = NK / 4;
                    if (n == 0 && i % kEvery == kEvery - 1 && i / kEvery < 3) lds_issue_row(lq, l4[i / kEvery + 1], sa, 32 * (i / kEvery + 1));
                    if (n == kN - 1) {
                        if (i + kAhead < NK) issue_first(NK + i + kAhead);
                        else issue_second(i + kAhead - NK);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    shadow(kDp + kN * i + n);
                }
            }
#pragma unroll
            for (int i = 0; i < 4 * NDB; ++i) {               // dV, then dK
                const int j = i % (2 * NDB), b2 = j / NDB, db = j % NDB;
                const bf16x8 f = lds_wait(lq, cf[i % kAhead]);
#pragma unroll
                for (int kb = 0; kb < kN; ++kb) {
                    if (i < 2 * NDB) mfma_acc(dv[kb][db], f, u32x4{pk[kb][4 * b2], pk[kb][4 * b2 + 1], pk[kb][4 * b2 + 2], pk[kb][4 * b2 + 3]});
                    else mfma_acc(dk[kb][db], f, u32x4{ds[kb][4 * b2], ds[kb][4 * b2 + 1], ds[kb][4 * b2 + 2], ds[kb][4 * b2 + 3]});
                    if (kb == kN - 1) {
                        if (i + kAhead < 4 * NDB) issue_second(i + kAhead);
                        const int n = i - (4 * NDB - 2 * kAhead);      // the next block's first fragments
                        if (n >= 0 && n < kAhead) lds_issue_row(lq, rf[n], next_row ^ (uint32_t)(n << 5), ib ? 0 : 32 * kRowBytes);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    shadow(kDv + kN * i + kb);
                }
            }
#pragma unroll
            for (int i = 0; i < kAhead; ++i) { lds_wait_raw(lq, rf[i]); rf[i].seq = 0; }
            __builtin_amdgcn_sched_barrier(0);
        };
        int stage = 0, it = 0;
        // Between the blocks of a step: the next tile is there for everybody, and the tile before this one has been read by
        // all; the one three steps ahead takes its place.
        auto turn = [&]() {
            // tile it + 1 precedes tile it + 2 in the (in-order) vmcnt queue
            if (it + 2 < n_iter) __builtin_amdgcn_s_waitcnt(0x0F70 | (kDmaPerStage & 15) | ((kDmaPerStage >> 4) << 14));     // vmcnt(kDmaPerStage)
            else __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            if (it + 3 < n_iter) dma_stage(stage == 0 ? kKwStages - 1 : stage - 1, true);
        };
        auto move_of = [&]() { return stage == kKwStages - 1 ? (uint32_t)(-(kKwStages - 1) * kKwStageBytes) : (uint32_t)kKwStageBytes; };
        auto advance = [&]() {
            const uint32_t move = move_of();
#pragma unroll
            for (int i = 0; i < 2 * NDB; ++i) fa_col[i] += move;
            fa_row += move;
            const bool last = stage == kKwStages - 1;
            stat += last ? (uint32_t)(-(kKwStages - 1) * 2 * kKwBM * 4) : (uint32_t)(2 * kKwBM * 4);
            stage = last ? 0 : stage + 1;
            ++it;
        };
        // Three loops: tiles before the wave's keys, the tile of its diagonal, the others.  One loop with a choice of bodies
        // would have the accumulators meet in vector registers; so they stay in their file from one to the next.
        const int skip = active ? min(max(td - qt_first, 0) * G, n_iter) : n_iter;
        const int diag = active ? min(max(td + 1 - qt_first, 0) * G, n_iter) : n_iter;
        while (it < skip) { turn(); advance(); }
        if (it < n_iter) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                LdsQueue lq{0};
                lds_issue_row(lq, rf[i], fa_row ^ (uint32_t)(i << 5), 0);
                lds_wait_raw(lq, rf[i]);
                rf[i].seq = 0;
            }
        }
        keep_acc(dv, dk);
        while (it < diag) {
            block(std::integral_constant<int, 1>{}, std::true_type{}, 0, fa_row);
            turn();
            block(std::integral_constant<int, 2>{}, std::true_type{}, 1, fa_row + move_of());
            advance();
        }
        keep_acc(dv, dk);
        while (it < n_iter) {
            block(std::integral_constant<int, 2>{}, std::false_type{}, 0, fa_row);
            turn();
            block(std::integral_constant<int, 2>{}, std::false_type{}, 1, fa_row + move_of());
            advance();
        }
        keep_acc(dv, dk);
        __builtin_amdgcn_s_barrier();                         // every wave is done with the ring
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");    // the last products are there
        if (!short_item) wf.claim(list.hm, list.cursors);
        if (active) {
            const uint32_t o_stage = lds0 + (uint32_t)(wave * 3 * 32 * kRowBytes);      // this wave's 24 KB of the ring
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                if (wkey0 + 32 * kb < L) {
                    const int64_t out = (int64_t)(row0 + wkey0 + 32 * kb) * kv_stride + (int64_t)g * D;
                    store_rows_via_lds<D>(p.dv + out, kv_stride, L - wkey0 - 32 * kb, dv[kb], unscale, o_stage, lane);
                    store_rows_via_lds<D>(p.dk + out, kv_stride, L - wkey0 - 32 * kb, dk[kb], p.scale * unscale, o_stage + 32 * kRowBytes, lane);
                }
            }
        }
        have = wf.next(list.hm, list.cursors, list.items, slot, wi);
    }
    if (p.tr.rec && *list.hdr > 0) trace_write(p.tr, 1, t_start, n_done);       // (a list may be left to the other form)
}

}  // namespace hyd
