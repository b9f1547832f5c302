// fp32 kernels: the same operation for fp32 inputs on v_mfma_f32_32x32x2_f32 (fp32 products and
// sums, tolerance 1e-5; 64 clocks for 2048 multiply-adds).  Work item = 64 query rows of one head
// (forward, dQ: 8 waves = 2 groups of 32 rows x 4 splits) or 32 keys of one KV head (dK/dV: 4
// waves = 4 splits): the other side of the product streams through LDS in tiles of 128 rows, each
// split takes its own 32-row block of every tile, and the splits are added up once per item.
//
// Why this split.  fp32 batches are small (a numerical check next to the bf16 path), so what a
// call takes is its longest item: splitting the streamed side over the waves of a workgroup makes
// that item 128 rows per step long instead of 32 or 64.  With 64-row tiles and two splits the
// 4001-token case below took 300 us in the forward, 414 us in dQ and 405 us in dK/dV.
//
// What bounds them is the matrix pipe: a 32x32 block of one product is D/2 instructions of 64
// clocks against D/8 16-byte or D/2 4-byte LDS reads per lane and 16 exponentials.  Loads of the next
// tile go out as soon as an operand tile has been used for the last time in a step, so that they
// run under the other operand's products and one LDS buffer per operand is enough.
// Measured (MI355X, forward / dQ / dK/dV; before: one thread per row with plain multiply-adds):
//   4001 tokens in 7 sequences, 8 heads, d = 128     172 / 233 / 302 us, before 6360 / 7001 / 38107 us
//   one sequence of 8192, 16 heads, d = 128          109 / 120 / 98 TFLOP/s of useful products
//                                                    (a large fp32 library product: 151)
#pragma once
#include <float.h>

#include "hyd_sched.h"

namespace hyd {

constexpr int kF32BM = 64, kF32KvBN = 32;        // rows of an item: forward and dQ; keys of an item: dK/dV
constexpr int kF32Splits = 4, kF32Tile = 32 * kF32Splits;      // rows of a streamed tile, a 32-row block for each split
constexpr int kF32Waves = 8, kF32KvWaves = 4;
template <int D> constexpr int f32_tile_bytes() { return kF32Tile * D * 4; }
template <int D> constexpr int f32_lds() { return 2 * f32_tile_bytes<D>() + 128; }      // two operand tiles, work slot, repeat flag

struct F32Params {
    const float* q; const float* k; const float* v; const float* o; const float* d_o;
    const float* lse_in; float* D;
    float* o_out; float* lse_out;
    float* dq; float* dk; float* dv;
    int T, hq, hkv;
    float scale;
    const int* hdr; int* cursors; const int* items;
    HeadMap hm;
    WgTrace tr;
};

// D[32][32] += A[32][2] * B[2][32]: lane l holds a = A[l % 32][l / 32], b = B[l / 32][l % 32]; the
// accumulator has the lane map of mfma32.
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// LDS tile: 128 rows of D floats, 16-byte chunk c of row r at chunk position c ^ (r & 15): 16 lanes
// reading one chunk of 16 consecutive rows hit 16 different positions.
//
// Operands.  The contraction order of a product is free as long as both operands agree, so step
// 4a + e of a product over the head dimension uses element 8a + 4 * half + e in half `half` of the
// wave: one 16-byte LDS read (`row`) or global read feeds four instructions.  In a product over
// tile rows, step r uses row 8 (r / 4) + 4 half + r % 4 of the 32-row block, which is the row that
// accumulator register r holds: P and dS are operands as they stand, and the other operand is a
// 4-byte read (`col`) of that row at column 32 db + lane % 32.
template <int D, int NW>
struct F32Lds {
    static constexpr int kRB = D * 4;                // bytes of a row
    uint32_t row[8], col[4];                         // of the split's 32-row block of a tile
    uint32_t voff[2];                                // direct-to-LDS loads, see load()
    int wave;
    __device__ __forceinline__ void init(int lane, int w, int split, const char* lds_base, uint32_t stride_b) {
        const int l32 = lane & 31, half = lane >> 5;
        const uint32_t base = (uint32_t)(uintptr_t)(lds_char*)lds_base + (uint32_t)(split * 32 * kRB);
#pragma unroll
        for (int a = 0; a < 8; ++a) row[a] = base + (uint32_t)(l32 * kRB + (((2 * a + half) ^ (l32 & 15)) << 4));
#pragma unroll
        for (int m = 0; m < 4; ++m)
            col[m] = base + (uint32_t)(4 * half * kRB + ((((l32 >> 2) ^ (4 * half + m)) & 7) << 4) + (l32 & 3) * 4);
        wave = w;
        // lane i of a 1 KB load fills chunk position i % (D/4) of row i / (D/4) of the instruction's rows
        constexpr int kCh = D / 4;
        const int r = (64 / kCh) * wave + lane / kCh, pos = lane % kCh;
        voff[0] = (uint32_t)r * stride_b + (uint32_t)((pos ^ (r & 15)) << 4);
        voff[1] = (uint32_t)r * stride_b + (uint32_t)((pos ^ ((r + 8) & 15)) << 4);
    }
    // one tile (row 0 = byte soff of the resource) to the LDS address of a tile
    static constexpr int kLoads = kF32Tile * D * 4 / 1024 / NW;         // instructions per wave
    __device__ __forceinline__ void load(const __amdgpu_buffer_rsrc_t& rs, char* lds, uint32_t soff, uint32_t stride_b) const {
        typedef __attribute__((address_space(3))) void lds_void_t;
        constexpr int kRows = 256 / D * NW;            // rows per group of NW instructions (one per wave): a multiple of 8
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(lds + (NW * j + wave) * 1024), 16, voff[(j * kRows / 8) & 1],
                                                     soff + (uint32_t)(j * kRows) * stride_b, 0, 0);
    }
    __device__ __forceinline__ f32x4 row4(int tile, int a) const {
        typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
        return *(lds_f32x4*)(uintptr_t)(row[a & 7] + (uint32_t)(tile + (a >> 3) * 256));
    }
    __device__ __forceinline__ float col1(int tile, int r, int db) const {
        typedef __attribute__((address_space(3))) const float lds_f32;
        const int c8 = (8 * db) ^ (8 * ((r >> 2) & 1));
        return *(lds_f32*)(uintptr_t)(col[r & 3] + (uint32_t)(tile + (8 * (r >> 2) + (r & 3)) * kRB + (c8 << 4)));
    }
};

// acc[32][32] += rows of the split's block of an LDS tile times the row held in x (32 x 32 block of a product over the head dimension)
template <int D, int NW>
__device__ __forceinline__ void f32_row_product(f32x16& acc, const F32Lds<D, NW>& fl, int tile, const f32x4 (&x)[D / 8]) {
    f32x4 f = fl.row4(tile, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < D / 8; ++a) {
        const f32x4 c = f;
        if (a + 1 < D / 8) f = fl.row4(tile, a + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma_f32(c[e], x[a][e], acc);
        __builtin_amdgcn_sched_barrier(0);
    }
}
// acc[db] += (block of an LDS tile, transposed) times the accumulator-shaped factor p.  The order is
// pinned with scheduling fences: left alone, the compiler puts every LDS read right before its
// use (read, wait, multiply), which doubled the time of the kernels.
template <int D, int NW>
__device__ __forceinline__ void f32_col_product(f32x16 (&acc)[D / 32], const F32Lds<D, NW>& fl, int tile, const f32x16& p) {
    constexpr int NDB = D / 32, kAhead = D == 128 ? 1 : 2, kBuf = kAhead + 1;       // steps read ahead: 4 MFMAs of 64 clocks
    float f[kBuf][NDB];
#pragma unroll
    for (int r = 0; r < kAhead; ++r)
#pragma unroll
        for (int db = 0; db < NDB; ++db) f[r][db] = fl.col1(tile, r, db);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (r + kAhead < 16) {
#pragma unroll
            for (int db = 0; db < NDB; ++db) f[(r + kAhead) % kBuf][db] = fl.col1(tile, r + kAhead, db);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < NDB; ++db) acc[db] = mfma_f32(f[r % kBuf][db], p[r], acc[db]);
        __builtin_amdgcn_sched_barrier(0);
    }
}
// exp(x) to fp32 accuracy: x log2(e) is formed as hi + lo (lo from the rounding error of the product and
// the rest of the constant), 2^hi by the hardware instruction, 2^lo = 1 + lo ln(2).  Down to x = -inf, where
// lo would not be a number (hence the maximum, which keeps a NaN); not for x above 88.7, which no visible pair has.
__device__ __forceinline__ float f32_exp(float x) {
    constexpr float kL2e = 1.44269504088896340736f, kL2eRest = 1.44269504088896340736 - (double)kL2e;
    constexpr float kLn2 = 0.69314718055994530942f;
    x = __builtin_elementwise_maximum(x, -200.f);
    const float hi = x * kL2e;
    const float lo = __builtin_fmaf(x, kL2eRest, __builtin_fmaf(x, kL2e, -hi));
    const float e = __builtin_amdgcn_exp2f(hi);
    return __builtin_fmaf(e, lo * kLn2, e);
}
template <int N> __device__ __forceinline__ void f32_zero(f32x16 (&a)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) a[i][r] = 0.f;
}
// the row of `lane` as the operand of f32_row_product: elements 8a + 4 half + {0..3}
template <int D>
__device__ __forceinline__ void f32_load_row(f32x4 (&x)[D / 8], const float* row, int half) {
#pragma unroll
    for (int a = 0; a < D / 8; ++a) x[a] = *reinterpret_cast<const f32x4*>(row + 8 * a + 4 * half);
}
// transposed accumulators -> the lane's row (element 32 db + 8 rq + 4 half + {0..3} in registers 4 rq ..)
template <int D>
__device__ __forceinline__ void f32_store_row(float* row, const f32x16 (&acc)[D / 32], float mul, int half) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            const f32x4 v = {acc[db][4 * rq] * mul, acc[db][4 * rq + 1] * mul, acc[db][4 * rq + 2] * mul, acc[db][4 * rq + 3] * mul};
            *reinterpret_cast<f32x4*>(row + 32 * db + 8 * rq + 4 * half) = v;
        }
}
// accumulators of the other splits through LDS (lane-major: conflict-free), for split 0 to add
template <int N>
__device__ __forceinline__ void f32_put(char* lds, const f32x16 (&a)[N], int lane) {
    f32x4* p = reinterpret_cast<f32x4*>(lds) + lane;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) p[(4 * i + q) * 64] = f32x4{a[i][4 * q], a[i][4 * q + 1], a[i][4 * q + 2], a[i][4 * q + 3]};
}
template <int N>
__device__ __forceinline__ void f32_add(f32x16 (&a)[N], float wa, const char* lds, float wb, int lane) {
    const f32x4* p = reinterpret_cast<const f32x4*>(lds) + lane;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = p[(4 * i + q) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[i][4 * q + e] = a[i][4 * q + e] * wa + v[e] * wb;
        }
}
// vmcnt(N) with everything else left alone, then the workgroup barrier
template <int N>
__device__ __forceinline__ void f32_arrive() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// LDS reads of this wave done, then the workgroup barrier (the tile may be overwritten)
__device__ __forceinline__ void f32_release() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- one row at a time
//
// Infinities and NaN.  A product over tile rows takes a hidden pair as 0 * x, which is none if x is not finite: a bad row of
// the streamed side would reach all 32 lanes of the block where some lanes see it and others do not (the
// diagonal one, and in dK/dV the one that runs past the sequence).  The tile loop does not look for that.  At the end of an
// item, a wave whose sums are not finite looks at those blocks, and if there is a bad row among them the
// workgroup takes the rows of the item again, pair by pair, visible pairs only.
//
// The functions below take one row: the wave's lanes hold its elements, D / 64 each, and the other side's rows follow one after
// the other, kU in flight.
template <int D> struct F32Part { float v[D / 64]; };
template <int D>
__device__ __forceinline__ F32Part<D> f32_part(const float* row, int lane) {
    F32Part<D> x;
#pragma unroll
    for (int e = 0; e < D / 64; ++e) x.v[e] = row[64 * e + lane];
    return x;
}
template <int D>
__device__ __forceinline__ float f32_part_dot(const F32Part<D>& a, const F32Part<D>& b) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < D / 64; ++e) s = __builtin_fmaf(a.v[e], b.v[e], s);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m, 64);
    return s;
}
template <int D>
__device__ __forceinline__ void f32_part_add(F32Part<D>& acc, float f, const F32Part<D>& x) {
#pragma unroll
    for (int e = 0; e < D / 64; ++e) acc.v[e] = __builtin_fmaf(f, x.v[e], acc.v[e]);
}
template <int D>
__device__ __forceinline__ void f32_part_store(float* row, const F32Part<D>& x, float mul, int lane) {
#pragma unroll
    for (int e = 0; e < D / 64; ++e) row[64 * e + lane] = x.v[e] * mul;
}
constexpr int kF32RowsU = 4;
// Sequences of up to kF32Short rows are taken this way from the start, a row per wave: an item of the tile path takes about 10 us
// however short it is.  The tile loops of the backward have no registers to spare at D = 128 (this path beside them
// costs 3 %), so there it is a kernel of its own, for batches that hold nothing longer.  Measured, 4096 sequences of one
// token, forward / backward in us, tile path -> this: 8 heads, d = 128 1202 / 3857 -> 337 / 517; 8/2 heads, d = 64 732 /
// 1700 -> 271 / 601; 1300 sequences of three tokens, 8 heads, d = 128 397 / 1266 -> 115 / 190.
constexpr int kF32Short = kF32Waves;
constexpr int f32_rows_lds() { return 128; }

template <int D>
__device__ __forceinline__ void f32_row_fwd(const F32Params& p, int row0, int i, int head, int lane) {
    asm volatile("" : "+v"(lane));           // (addresses are formed here: hoisted out of the item loop they spill registers in the tile loop)
    const int64_t at = ((int64_t)(row0 + i) * p.hq + head) * D, kv_stride = (int64_t)p.hkv * D;
    const int64_t kv = (int64_t)row0 * kv_stride + (int64_t)(head / (p.hq / p.hkv)) * D;
    const F32Part<D> q = f32_part<D>(p.q + at, lane);
    F32Part<D> o = {};
    float m = -INFINITY, l = 0.f;
    for (int j0 = 0; j0 <= i; j0 += kF32RowsU) {
        F32Part<D> k[kF32RowsU], v[kF32RowsU];
        float s[kF32RowsU];
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u) {
            const int64_t row = kv + min(j0 + u, i) * kv_stride;
            k[u] = f32_part<D>(p.k + row, lane);
            v[u] = f32_part<D>(p.v + row, lane);
        }
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u) s[u] = p.scale * f32_part_dot<D>(q, k[u]);
        float m_new = m;
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u) m_new = fmaxf(m_new, s[u]);        // (the row repeated past i changes nothing)
        const float ref = m_new == -INFINITY ? 0.f : m_new, alpha = f32_exp(m - ref);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) o.v[e] *= alpha;
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u)
            if (j0 + u <= i) {
                const float pr = f32_exp(s[u] - ref);
                l += pr;
                f32_part_add<D>(o, pr, v[u]);
            }
    }
    f32_part_store<D>(p.o_out + at, o, 1.f / l, lane);
    if (lane == 0) p.lse_out[(int64_t)head * p.T + row0 + i] = m + logf(l);
}

template <int D>
__device__ __forceinline__ void f32_row_dq(const F32Params& p, int row0, int i, int head, int lane) {
    asm volatile("" : "+v"(lane));           // (addresses are formed here: hoisted out of the item loop they spill registers in the tile loop)
    const int64_t at = ((int64_t)(row0 + i) * p.hq + head) * D, st = (int64_t)head * p.T + row0 + i, kv_stride = (int64_t)p.hkv * D;
    const int64_t kv = (int64_t)row0 * kv_stride + (int64_t)(head / (p.hq / p.hkv)) * D;
    const F32Part<D> q = f32_part<D>(p.q + at, lane), g = f32_part<D>(p.d_o + at, lane);
    const float Di = f32_part_dot<D>(f32_part<D>(p.o + at, lane), g), lse = p.lse_in[st];
    if (lane == 0) p.D[st] = Di;
    F32Part<D> acc = {};
    for (int j0 = 0; j0 <= i; j0 += kF32RowsU) {
        F32Part<D> k[kF32RowsU];
        float s[kF32RowsU], dp[kF32RowsU];
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u) {
            const int64_t row = kv + min(j0 + u, i) * kv_stride;
            k[u] = f32_part<D>(p.k + row, lane);
            s[u] = f32_part_dot<D>(q, k[u]);
            dp[u] = f32_part_dot<D>(g, f32_part<D>(p.v + row, lane));
        }
#pragma unroll
        for (int u = 0; u < kF32RowsU; ++u)
            if (j0 + u <= i) f32_part_add<D>(acc, f32_exp(__builtin_fmaf(p.scale, s[u], -lse)) * (dp[u] - Di), k[u]);
    }
    f32_part_store<D>(p.dq + at, acc, p.scale, lane);
}

template <int D>
__device__ __forceinline__ void f32_row_dkdv(const F32Params& p, int row0, int L, int j, int g, int lane) {
    asm volatile("" : "+v"(lane));           // (addresses are formed here: hoisted out of the item loop they spill registers in the tile loop)
    const int G = p.hq / p.hkv;
    const int64_t at = ((int64_t)(row0 + j) * p.hkv + g) * D, q_stride = (int64_t)p.hq * D;
    const F32Part<D> k = f32_part<D>(p.k + at, lane), v = f32_part<D>(p.v + at, lane);
    F32Part<D> dk = {}, dv = {};
    for (int h = g * G; h < (g + 1) * G; ++h)
        for (int i0 = j; i0 < L; i0 += kF32RowsU) {
            F32Part<D> q[kF32RowsU], d_o[kF32RowsU];
            float s[kF32RowsU], dp[kF32RowsU], lse[kF32RowsU], Di[kF32RowsU];
#pragma unroll
            for (int u = 0; u < kF32RowsU; ++u) {
                const int i = min(i0 + u, L - 1);
                const int64_t row = (int64_t)(row0 + i) * q_stride + (int64_t)h * D, st = (int64_t)h * p.T + row0 + i;
                q[u] = f32_part<D>(p.q + row, lane);
                d_o[u] = f32_part<D>(p.d_o + row, lane);
                s[u] = f32_part_dot<D>(q[u], k);
                dp[u] = f32_part_dot<D>(d_o[u], v);
                lse[u] = p.lse_in[st];
                Di[u] = p.D[st];
            }
#pragma unroll
            for (int u = 0; u < kF32RowsU; ++u)
                if (i0 + u < L) {
                    const float pr = f32_exp(__builtin_fmaf(p.scale, s[u], -lse[u]));
                    f32_part_add<D>(dv, pr, d_o[u]);
                    f32_part_add<D>(dk, pr * (dp[u] - Di[u]), q[u]);
                }
        }
    f32_part_store<D>(p.dk + at, dk, p.scale, lane);
    f32_part_store<D>(p.dv + at, dv, 1.f, lane);
}

template <int N>
__device__ __forceinline__ bool f32_all_finite(const f32x16 (&acc)[N]) {
    float z = 0.f;                                               // (these maxima keep a NaN)
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2) z = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(acc[i][r]), fabsf(acc[i][r + 1])), z);
    return !__any(!(z <= FLT_MAX));
}
// rows [first, min(first + 32, L)) of a tensor [.][stride] from `base` hold finite values only
template <int D>
__device__ __forceinline__ bool f32_rows_finite(const float* base, int64_t stride, int first, int L, int lane) {
    asm volatile("" : "+v"(lane));           // (addresses are formed here: hoisted out of the item loop they spill registers in the tile loop)
    float z = 0.f;
#pragma unroll 1
    for (int r = first; r < min(first + 32, L); ++r) {
        const F32Part<D> x = f32_part<D>(base + r * stride, lane);
#pragma unroll
        for (int e = 0; e < D / 64; ++e) z = __builtin_fmaf(x.v[e], 0.f, z);
    }
    return !__any(z != 0.f);
}

// Forward.  S^T[key][q] = K Q^T (one query row per lane), O^T[d][q] += V^T P^T.
// kSelf: one item per workgroup, found by itself (see SelfSchedule).
template <int D, bool kSelf>
__device__ __forceinline__ void fwd_fp32_items(const F32Params& p, const SelfSchedule* ss, char* smem) {
    constexpr int kT = f32_tile_bytes<D>(), NDB = D / 32, kL = F32Lds<D, kF32Waves>::kLoads;
    constexpr int kAcc = NDB * 64 * 64;                          // bytes of a wave's accumulators
    int* slot = reinterpret_cast<int*>(smem + 2 * kT);
    volatile int* bad = slot + kSlotInts;                        // see "one row at a time"
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave & 1, split = wave >> 1, l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const uint32_t stride_b = (uint32_t)p.hkv * D * 4;
    F32Lds<D, kF32Waves> fl;
    fl.init(lane, wave, split, smem, stride_b);
    WorkFetcher wf;
    WorkItem wi;
    auto claim = [&]() { if (!kSelf) wf.claim(p.hm, p.cursors); };
    bool have;
    if constexpr (kSelf) have = self_first(*ss, smem, 64 * kF32Waves, wi);
    else have = wf.first(p.hm, p.hdr, p.cursors, p.items, slot, wi, blockIdx.x);
    for (; have; have = kSelf ? false : wf.next(p.hm, p.cursors, p.items, slot, wi)) {
        const int head = wi.head, row0 = wi.row0, L = wi.len;
        bool rows = L <= kF32Short;
        if (rows) {
            claim();
        } else {
            const int q0 = (wi.lev - 1) * kF32BM, kv_end = min(L, q0 + kF32BM), n_kt = (kv_end + kF32Tile - 1) / kF32Tile;
            const int g = head / G, wrow0 = q0 + 32 * rg, i = wrow0 + l32;
            const uint32_t kv_bytes = (uint32_t)(kv_end - 1) * stride_b + D * 4;
            const __amdgpu_buffer_rsrc_t rk = make_rsrc(p.k + ((int64_t)row0 * p.hkv + g) * D, kv_bytes);
            const __amdgpu_buffer_rsrc_t rv = make_rsrc(p.v + ((int64_t)row0 * p.hkv + g) * D, kv_bytes);
            fl.load(rk, smem, 0, stride_b);
            f32x4 q[D / 8];
            f32_load_row<D>(q, p.q + ((int64_t)(row0 + min(i, L - 1)) * p.hq + head) * D, half);
            fl.load(rv, smem + kT, 0, stride_b);
            f32x16 o[NDB];
            f32_zero(o);
            if (tid == 0) *bad = 0;
            float m = -INFINITY, l = 0.f;
            for (int t = 0; t < n_kt; ++t) {
                const uint32_t nxt = (uint32_t)(t + 1) * kF32Tile * stride_b;
                const bool more = t + 1 < n_kt;
                if (t == max(n_kt - 2, 0)) claim();
                const int key0 = t * kF32Tile + 32 * split;
                const bool work = key0 <= wrow0 && wrow0 < L;        // else the block is hidden from all rows of the wave
                f32_arrive<kL>();                                    // K tile t is there
                f32x16 s[1];
                f32_zero(s);
                if (work) f32_row_product(s[0], fl, 0, q);
                f32_release();
                if (more) fl.load(rk, smem, nxt, stride_b);
                if (work) {
                    const int rel = i - key0 - 4 * half;             // register r is visible iff its key offset <= rel
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[0][r] *= p.scale;
                    if (key0 == wrow0) {                             // the diagonal block
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (8 * (r >> 2) + (r & 3) > rel) s[0][r] = -INFINITY;
                    }
                    float mx = s[0][0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[0][r]);
                    float lo, hi;
                    both_halves(mx, lo, hi);
                    const float m_new = fmaxf(m, fmaxf(lo, hi));
                    // (a row that has seen no score but -inf yet: every probability is 0)
                    const float ref = m_new == -INFINITY ? 0.f : m_new;
                    const float alpha = f32_exp(m - ref);
                    m = m_new;
                    float sum = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) { s[0][r] = f32_exp(s[0][r] - ref); sum += s[0][r]; }
                    l = l * alpha + sum;
                    if (__any(alpha != 1.f)) {
#pragma unroll
                        for (int db = 0; db < NDB; ++db)
#pragma unroll
                            for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
                    }
                }
                if (more) f32_arrive<kL>(); else f32_arrive<0>();    // V tile t is there
                if (work) f32_col_product(o, fl, kT, s[0]);
                f32_release();
                if (more) fl.load(rv, smem + kT, nxt, stride_b);
            }
            {   // l is still split over the two halves of the wave
                float lo, hi;
                both_halves(l, lo, hi);
                l = lo + hi;
            }
            // The splits' results meet in LDS: accumulators of split s > 0 and row group rg at 2 (s - 1) + rg,
            // (m, l) of every wave in the bytes behind them (the last quarter of the second tile).
            float* ml = reinterpret_cast<float*>(smem + 2 * kT - kAcc);
            if (split) f32_put(smem + (2 * (split - 1) + rg) * kAcc, o, lane);
            ml[wave * 128 + lane] = m;
            ml[wave * 128 + 64 + lane] = l;
            if (split == ((wrow0 >> 5) & (kF32Splits - 1)) && wrow0 < L && __builtin_expect(!f32_all_finite(o), 0))
                if (!f32_rows_finite<D>(p.v + ((int64_t)row0 * p.hkv + g) * D, (int64_t)p.hkv * D, wrow0, L, lane)) *bad = 1;
            __syncthreads();
            if (split == 0 && wrow0 < L) {
                float mt = m, lt = 0.f;                              // (a split that saw no key has m = -inf and l = 0)
#pragma unroll
                for (int x = 1; x < kF32Splits; ++x) mt = fmaxf(mt, ml[(2 * x + rg) * 128 + lane]);
                float w = f32_exp(m - mt);
                lt = l * w;
#pragma unroll
                for (int x = 1; x < kF32Splits; ++x) {
                    const float wx = f32_exp(ml[(2 * x + rg) * 128 + lane] - mt);
                    lt += ml[(2 * x + rg) * 128 + 64 + lane] * wx;
                    f32_add(o, w, smem + (2 * (x - 1) + rg) * kAcc, wx, lane);
                    w = 1.f;
                }
                if (i < L) {
                    f32_store_row<D>(p.o_out + ((int64_t)(row0 + i) * p.hq + head) * D, o, 1.f / lt, half);
                    if (half == 0) p.lse_out[(int64_t)head * p.T + row0 + i] = mt + logf(lt);
                }
            }
            rows = *bad != 0;
            if (__builtin_expect(rows, 0)) __syncthreads();      // the rows' stores above come first
        }
        if (__builtin_expect(rows, 0)) {
            for (int r = (wi.lev - 1) * kF32BM + wave; r < min(L, wi.lev * kF32BM); r += kF32Waves) f32_row_fwd<D>(p, row0, r, head, lane);
        }
    }
}

template <int D>
__global__ void __launch_bounds__(64 * kF32Waves, 1) hyd_fwd_fp32_kernel(F32Params p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    fwd_fp32_items<D, false>(p, nullptr, smem);
}
template <int D>
__global__ void __launch_bounds__(64 * kF32Waves, 1) hyd_fwd_self_fp32_kernel(F32Params p, SelfSchedule ss) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    fwd_fp32_items<D, true>(p, &ss, smem);
}

// dQ.  S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T.  Also forms D = rowsum(dO * O) of its rows, which
// the dK/dV kernel that follows reads.
template <int D, bool kRows, bool kSelf>
__device__ __forceinline__ void dq_fp32_items(const F32Params& p, const SelfSchedule* ss, char* smem) {
    constexpr int kT = f32_tile_bytes<D>(), NDB = D / 32, kL = F32Lds<D, kF32Waves>::kLoads;
    constexpr int kAcc = NDB * 64 * 64;
    int* slot = reinterpret_cast<int*>(smem + (kRows ? 0 : 2 * kT));
    volatile int* bad = slot + kSlotInts;                        // see "one row at a time"
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave & 1, split = wave >> 1, l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const uint32_t stride_b = (uint32_t)p.hkv * D * 4;
    F32Lds<D, kF32Waves> fl;
    fl.init(lane, wave, split, smem, stride_b);
    WorkFetcher wf;
    WorkItem wi;
    auto claim = [&]() { if (!kSelf) wf.claim(p.hm, p.cursors); };
    bool have;
    if constexpr (kSelf) have = self_first(*ss, smem, 64 * kF32Waves, wi);
    else have = wf.first(p.hm, p.hdr, p.cursors, p.items, slot, wi, blockIdx.x);
    for (; have; have = kSelf ? false : wf.next(p.hm, p.cursors, p.items, slot, wi)) {
        const int head = wi.head, row0 = wi.row0, L = wi.len;
        bool rows = kRows || (D == 64 && L <= kF32Short);
        if (rows) {
            claim();
        } else {
            const int q0 = (wi.lev - 1) * kF32BM, kv_end = min(L, q0 + kF32BM), n_kt = (kv_end + kF32Tile - 1) / kF32Tile;
            const int g = head / G, wrow0 = q0 + 32 * rg, i = wrow0 + l32, ic = min(i, L - 1);
            const uint32_t kv_bytes = (uint32_t)(kv_end - 1) * stride_b + D * 4;
            const __amdgpu_buffer_rsrc_t rk = make_rsrc(p.k + ((int64_t)row0 * p.hkv + g) * D, kv_bytes);
            const __amdgpu_buffer_rsrc_t rv = make_rsrc(p.v + ((int64_t)row0 * p.hkv + g) * D, kv_bytes);
            const int64_t roff = ((int64_t)(row0 + ic) * p.hq + head) * D, at = (int64_t)head * p.T + row0 + ic;
            fl.load(rk, smem, 0, stride_b);
            f32x4 q[D / 8], dof[D / 8];
            f32_load_row<D>(q, p.q + roff, half);
            f32_load_row<D>(dof, p.d_o + roff, half);
            float Di = 0.f;
#pragma unroll
            for (int a = 0; a < D / 8; ++a) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(p.o + roff + 8 * a + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) Di = __builtin_fmaf(x[e], dof[a][e], Di);
            }
            {
                float lo, hi;
                both_halves(Di, lo, hi);
                Di = lo + hi;
            }
            if (split == 0 && half == 0 && i < L) p.D[at] = Di;
            const float lse = p.lse_in[at];
            fl.load(rv, smem + kT, 0, stride_b);
            f32x16 acc[NDB];
            f32_zero(acc);
            if (tid == 0) *bad = 0;
            for (int t = 0; t < n_kt; ++t) {
                const uint32_t nxt = (uint32_t)(t + 1) * kF32Tile * stride_b;
                const bool more = t + 1 < n_kt;
                if (t == max(n_kt - 2, 0)) claim();
                const int key0 = t * kF32Tile + 32 * split;
                const bool work = key0 <= wrow0 && wrow0 < L;
                f32x16 s[1], dp[1];
                f32_zero(s);
                f32_zero(dp);
                if (t == 0) f32_arrive<kL>(); else f32_arrive<0>();  // K tile t (from the second tile on V was requested first)
                if (work) f32_row_product(s[0], fl, 0, q);
                if (t == 0) f32_arrive<0>();                         // V tile t
                if (work) f32_row_product(dp[0], fl, kT, dof);
                f32_release();
                if (more) fl.load(rv, smem + kT, nxt, stride_b);
                if (work) {
                    const int rel = i - key0 - 4 * half;
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[0][r] = f32_exp(__builtin_fmaf(p.scale, s[0][r], -lse)) * (dp[0][r] - Di);
                    if (key0 == wrow0) {                             // the diagonal block
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (8 * (r >> 2) + (r & 3) > rel) s[0][r] = 0.f;
                    }
                    f32_col_product(acc, fl, 0, s[0]);
                }
                f32_release();
                if (more) fl.load(rk, smem, nxt, stride_b);
            }
            if (split) f32_put(smem + (2 * (split - 1) + rg) * kAcc, acc, lane);
            if (split == ((wrow0 >> 5) & (kF32Splits - 1)) && wrow0 < L && __builtin_expect(!f32_all_finite(acc), 0))
                if (!f32_rows_finite<D>(p.k + ((int64_t)row0 * p.hkv + g) * D, (int64_t)p.hkv * D, wrow0, L, lane)) *bad = 1;
            __syncthreads();
            if (split == 0 && wrow0 < L) {
#pragma unroll
                for (int x = 1; x < kF32Splits; ++x) f32_add(acc, 1.f, smem + (2 * (x - 1) + rg) * kAcc, 1.f, lane);
                if (i < L) f32_store_row<D>(p.dq + roff, acc, p.scale, half);
            }
            rows = *bad != 0;
            if (__builtin_expect(rows, 0)) __syncthreads();      // the rows' stores above come first
        }
        if (__builtin_expect(rows, 0)) {
            for (int r = (wi.lev - 1) * kF32BM + wave; r < min(L, wi.lev * kF32BM); r += kF32Waves) f32_row_dq<D>(p, row0, r, head, lane);
        }
    }
}

template <int D, bool kRows = false>
__global__ void __launch_bounds__(64 * kF32Waves, 1) hyd_bwd_dq_fp32_kernel(F32Params p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    dq_fp32_items<D, kRows, false>(p, nullptr, smem);
}
// (builds the list of the dK/dV kernel that follows, besides its own)
template <int D>
__global__ void __launch_bounds__(64 * kF32Waves, 1) hyd_bwd_dq_self_fp32_kernel(F32Params p, SelfSchedule ss) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    dq_fp32_items<D, false, true>(p, &ss, smem);
}

// dK/dV.  S[i][j] = Q K^T and dP[i][j] = dO V^T (one key per lane), dV^T += dO^T P, dK^T += Q^T dS.  K and V
// rows of the item stay in registers next to both accumulator sets; that takes more than 256
// registers, so one wave per SIMD.
template <int D, bool kRows = false>
__global__ void __launch_bounds__(64 * kF32KvWaves, 1) hyd_bwd_dkdv_fp32_kernel(F32Params p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int kT = f32_tile_bytes<D>(), NDB = D / 32;
    constexpr int kAcc = NDB * 64 * 64;
    int* slot = reinterpret_cast<int*>(smem + (kRows ? 0 : 2 * kT));
    volatile int* bad = slot + kSlotInts;                        // see "one row at a time"
    const int tid = threadIdx.x, lane = tid & 63;
    const int split = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int G = p.hq / p.hkv;
    const uint32_t stride_b = (uint32_t)p.hq * D * 4;
    F32Lds<D, kF32KvWaves> fl;
    fl.init(lane, split, split, smem, stride_b);
    WorkFetcher wf;
    WorkItem wi;
    for (bool have = wf.first(p.hm, p.hdr, p.cursors, p.items, slot, wi, blockIdx.x); have; have = wf.next(p.hm, p.cursors, p.items, slot, wi)) {
        const int g = wi.head, row0 = wi.row0, L = wi.len;
        bool rows = kRows || (D == 64 && L <= kF32Short);
        if (rows) {
            wf.claim(p.hm, p.cursors);
        } else {
            const int j0 = ((L + kF32KvBN - 1) / kF32KvBN - wi.lev) * kF32KvBN, j = j0 + l32;
            const int64_t koff = ((int64_t)(row0 + min(j, L - 1)) * p.hkv + g) * D;
            const uint32_t q_bytes = (uint32_t)(L - 1) * stride_b + D * 4;
            // iterations: tiles of query rows from j0 on outer, the group's heads inner
            int ld_i = j0, ld_h = 0;
            auto load_q = [&]() {
                fl.load(make_rsrc(p.q + ((int64_t)row0 * p.hq + g * G + ld_h) * D, q_bytes), smem, (uint32_t)ld_i * stride_b, stride_b);
            };
            auto load_do = [&]() {                                   // follows load_q of the same iteration
                fl.load(make_rsrc(p.d_o + ((int64_t)row0 * p.hq + g * G + ld_h) * D, q_bytes), smem + kT, (uint32_t)ld_i * stride_b, stride_b);
                if (++ld_h == G) { ld_h = 0; ld_i += kF32Tile; }
            };
            load_q();
            f32x4 kr[D / 8], vr[D / 8];
            f32_load_row<D>(kr, p.k + koff, half);
            f32_load_row<D>(vr, p.v + koff, half);
            load_do();
            f32x16 acck[NDB], accv[NDB];
            f32_zero(acck);
            f32_zero(accv);
            if (tid == 0) *bad = 0;
            const int n_iter = (L - j0 + kF32Tile - 1) / kF32Tile * G;
            int ti = j0, hh = 0;
            for (int it = 0; it < n_iter; ++it) {
                const bool more = it + 1 < n_iter;
                if (it == max(n_iter - 2, 0)) wf.claim(p.hm, p.cursors);
                const int i0 = ti + 32 * split;
                const bool work = i0 < L;
                // statistics of the block's rows (register r: row i0 + 8 (r / 4) + 4 half + r % 4); rows past the
                // sequence repeat its last one and are masked below, as exp(-LSE) need not be finite
                float nl[16], nd[16];
                if (work) {
                    const int64_t at = (int64_t)(g * G + hh) * p.T + row0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int ii = min(i0 + 8 * (r >> 2) + 4 * half + (r & 3), L - 1);
                        nl[r] = p.lse_in[at + ii];
                        nd[r] = p.D[at + ii];
                    }
                }
                f32x16 s[1], dp[1];
                f32_zero(s);
                f32_zero(dp);
                f32_arrive<0>();                                     // Q and dO tiles of this iteration
                if (work) {
                    f32_row_product(s[0], fl, 0, kr);
                    f32_row_product(dp[0], fl, kT, vr);
                    // register r is visible iff its row offset is in [rel, end): from the key on, inside the sequence
                    const int rel = j - i0 - 4 * half, end = L - i0 - 4 * half;
                    const bool part = i0 == j0 || i0 + 32 > L;       // else the whole block is
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = 8 * (r >> 2) + (r & 3);
                        float pr = f32_exp(__builtin_fmaf(p.scale, s[0][r], -nl[r]));
                        float ds = pr * (dp[0][r] - nd[r]);
                        if (part) {
                            pr = row >= rel && row < end ? pr : 0.f;
                            ds = row >= rel && row < end ? ds : 0.f;
                        }
                        s[0][r] = pr;
                        dp[0][r] = ds;
                    }
                    f32_col_product(acck, fl, 0, dp[0]);
                }
                f32_release();
                if (more) load_q();                                  // under the dV product
                if (work) f32_col_product(accv, fl, kT, s[0]);
                f32_release();
                if (more) load_do();
                if (++hh == G) { hh = 0; ti += kF32Tile; }
            }
            if (split) {
                f32_put(smem + 2 * (split - 1) * kAcc, acck, lane);
                f32_put(smem + (2 * (split - 1) + 1) * kAcc, accv, lane);
            }
            if (__builtin_expect(!f32_all_finite(acck) || !f32_all_finite(accv), 0)) {
                const int last = j0 + (L - 1 - j0) / 32 * 32;        // the blocks in question: split 0's first, and the last one
                bool finite = true;
                for (int h = 0; h < G; ++h) {
                    const int64_t q_stride = (int64_t)p.hq * D, at = ((int64_t)row0 * p.hq + g * G + h) * D;
                    if (split == 0) finite = finite && f32_rows_finite<D>(p.q + at, q_stride, j0, L, lane) && f32_rows_finite<D>(p.d_o + at, q_stride, j0, L, lane);
                    if (((last - j0) / 32) % kF32Splits == split)
                        finite = finite && f32_rows_finite<D>(p.q + at, q_stride, last, L, lane) && f32_rows_finite<D>(p.d_o + at, q_stride, last, L, lane);
                }
                if (!finite) *bad = 1;
            }
            __syncthreads();
            if (split == 0) {
#pragma unroll
                for (int x = 0; x < kF32Splits - 1; ++x) {
                    f32_add(acck, 1.f, smem + 2 * x * kAcc, 1.f, lane);
                    f32_add(accv, 1.f, smem + (2 * x + 1) * kAcc, 1.f, lane);
                }
                if (j < L) {
                    f32_store_row<D>(p.dk + koff, acck, p.scale, half);
                    f32_store_row<D>(p.dv + koff, accv, 1.f, half);
                }
            }
            rows = *bad != 0;
            if (__builtin_expect(rows, 0)) __syncthreads();      // the rows' stores above come first
        }
        if (__builtin_expect(rows, 0)) {
            const int j0 = ((L + kF32KvBN - 1) / kF32KvBN - wi.lev) * kF32KvBN;
            for (int r = j0 + split; r < min(L, j0 + kF32KvBN); r += kF32KvWaves) f32_row_dkdv<D>(p, row0, L, r, g, lane);
        }
    }
}

}  // namespace hyd
