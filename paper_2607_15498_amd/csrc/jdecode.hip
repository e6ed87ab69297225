// Decode over the shared cross-head basis (Sec. 3.1 Eq. (1) "Joint per-token vector" and "Shared
// basis"; Eq. (6)), gfx950: q [S][Q][H][d], at most 32 query rows (Q H) per sequence.
//
//   jq_kernel  q'_row = W_K,g q_row / sqrt(d) (fp32, [S][NQ][R]); further workgroups attend to the
//              exact rows (window and appended tokens), one per query row, original space;
//   js_kernel  scores of 128 tokens at a time, streamed through an LDS ring; wave = a slice of 128
//              coefficients of a tile of 16 tokens, the slices' partial scores summed in order
//              through LDS; scores [token][NQ] and a record (max, sum of exponentials) per block;
//   jv_kernel  rank-space value sums in the frame of all blocks' maximum: a workgroup takes two
//              slices (i and last - i, whose row counts together vary least) of a range of tokens
//              and only the rows that exist: slice s has one for every token that keeps more than
//              128 s (13% padding; 16 consecutive tokens at their largest rank cost 2.5 times the
//              kept coefficients);
//   jc_kernel  the ranges' sums added in order and rotated back with W_V,g^T, per (g, 32
//              coefficients);
//   jo_kernel  these parts added in order, the exact part added, division by the sum.
//
// Scores and values are two launches because a single pass leaves a record of NQ x R sums per
// workgroup, 33.5 MB to write and read back for 26.7 MB of coefficients; values over 64 ranges
// leave 8 MB, and the second read of the coefficients comes from the last-level cache.
// Llama layer, 32768 tokens, R = 1024: 49.7 us the call, the launches 6.2 + 18.2 + 18.9 + 5.0 +
// 3.8 us in a kernel trace (which closes no gaps: they need not add up to the call); the single pass
// (47.7 us in the trace, 16 consecutive tokens per step, one step's loads ahead) with its q', exact
// and three combining launches took 74.6 us the call.
#include <type_traits>

#include "vr_gemm.h"
#include "vr_internal.h"

namespace vr {

constexpr int JSEQ = 16;              // sequences per launch
constexpr int JROWS = 32;             // query rows per sequence at most (two 16-row tiles)
constexpr int JSL = 128;              // coefficients per slice
constexpr int JX_CAP = 8192;          // exact slots the exact workgroups hold in LDS
constexpr int JS_T = 1024, JS_B = 128;  // score workgroup: threads, tokens per block at most
constexpr int JV_T = 1024, JV_B = 512;  // value workgroup: threads, tokens per block of its range
constexpr int JC_K = 32;              // coefficients per rotation workgroup

struct JSeq {
    const void* coef;
    const uint32_t* offset;
    const void* kx;
    const void* vx;
    const void* q;
    void* out;
    int64_t n_exact;
};

struct JDec {
    JSeq seq[JSEQ];
    const float* W;
    u32x4* qf;      // [seq][R / 32][NQ / 16][hi, lo][64] q' / sqrt(d) as MFMA fragments
    float* S;       // [seq][bt n_blk][NQ] scores
    float* ml;      // [seq][n_blk][2][NQ] max and sum of exponentials per block of tokens
    float* rec;     // [seq][n_sp][NQ][R] value sums per range of tokens
    float* xrec;    // [seq][rows][2 + 128]: m, l, acc of the exact rows
    float* part;    // [seq][G][R / 32][rows of one g][128] rotated parts
    int64_t N, cap;
    int G, H, hpg, rows, nr, NQ, R, ns;
    int bt, n_blk, s_wg;    // tokens per block, blocks and score workgroups per sequence
    int n_sp, tps;          // ranges and tokens per range, per sequence
};

__device__ __forceinline__ float jd_wave_max(float v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float jd_wave_sum(float v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// 8 consecutive elements from a 16-byte aligned address as fp32
template <bool F32>
__device__ __forceinline__ void ld8(const void* base, int64_t at, float (&x)[8]) {
    if constexpr (F32) {
        const f32x4 a = ld4((const float*)base + at), b = ld4((const float*)base + at + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
    } else {
        const u32x4 a = load16((const uint16_t*)base + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[2 * e] = bf_lo(a[e]); x[2 * e + 1] = bf_hi(a[e]); }
    }
}

// 8 consecutive stored coefficients at any element index, raw (bf16: 4 words, fp32: 8)
template <bool F32> struct Raw8 { u32x4 w[F32 ? 2 : 1]; };
template <bool F32>
__device__ __forceinline__ Raw8<F32> ld_raw8(const void* coef, uint32_t at) {
    Raw8<F32> r;
    const uint8_t* p = (const uint8_t*)coef + (uint64_t)at * (F32 ? 4 : 2);
#pragma unroll
    for (int i = 0; i < (F32 ? 2 : 1); ++i) __builtin_memcpy(&r.w[i], p + 16 * i, 16);
    return r;
}
// the first nv (0..8) of them as bf16 fragments (fp32: hi and lo), the rest 0
template <bool F32>
__device__ __forceinline__ void frag8(const Raw8<F32>& r, int nv, u32x4& hi, u32x4& lo) {
    if constexpr (F32) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = e < nv ? __uint_as_float(r.w[e >> 2][e & 3]) : 0.f;
        split8(x, hi, lo);
    } else {
        hi = keep_first(r.w[0], nv);
    }
}

typedef __attribute__((address_space(3))) uint8_t jd_lds;
// waits until at most n (wave-uniform, >= 0; more than 8 counts as 8) of this wave's loads are in flight
__device__ __forceinline__ void jd_wait(int n) {
    switch (n) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
        case 7: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    }
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(const jd_lds*)p);
}

// ---- q' and the exact rows ------------------------------------------------------------------
// Workgroups [0, ns rows): one per (sequence, query row), the exact rows.  The others: one per
// (sequence, g, 32 coefficients), q' for all of head g's rows; 8 threads per coefficient with 16
// dims each, whole 128-byte lines of W per load.  Both are latency: every load issues at once.
template <bool F32>
__global__ __launch_bounds__(256) void jq_kernel(JDec p) {
    typedef typename std::conditional<F32, float, uint16_t>::type ET;
    __shared__ __attribute__((aligned(16))) float xs[JX_CAP];
    __shared__ __attribute__((aligned(16))) float red[16][D];
    __shared__ float wred[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int b = blockIdx.x;
    if (b >= p.ns * p.rows) {
        b -= p.ns * p.rows;
        const int kb_n = p.R / 32;
        const int s = b / (p.G * kb_n), g = b / kb_n % p.G, kb = b % kb_n;
        const int k = kb * 32 + (tid >> 3), pt = tid & 7;
        const float* w = p.W + (int64_t)k * (2 * p.G * D) + g * D;
        f32x4 wv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) wv[c] = ld4(w + 4 * (pt + 8 * c));
        // head g's query rows (row r: query r / hpg, head g hpg + r % hpg) as fp32
        for (int i = tid; i < p.nr * 16; i += 256) {
            const int r = i >> 4, c = i & 15;
            float x[8];
            ld8<F32>(p.seq[s].q, ((int64_t)(r / p.hpg) * p.H + g * p.hpg + r % p.hpg) * D + 8 * c, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) xs[r * D + 8 * c + e] = x[e];
        }
        __syncthreads();
        for (int r = 0; r < p.nr; ++r) {
            float a = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 x = ld4(&xs[r * D + 4 * (pt + 8 * c)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) a = fmaf(wv[c][e], x[e], a);
            }
            a += __shfl_xor(a, 1, 64);
            a += __shfl_xor(a, 2, 64);
            a += __shfl_xor(a, 4, 64);
            if (pt == 0) red[r >> 2][(r & 3) * 32 + (tid >> 3)] = a * 0.08838834764831845f;
        }
        __syncthreads();
        // 8 coefficients of one row per thread, as that row's lane of the step's fragment
        for (int i = tid; i < p.nr * 4; i += 256) {
            const int r = i >> 2, grp = i & 3, row = (r / p.hpg) * p.H + g * p.hpg + r % p.hpg;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = red[r >> 2][(r & 3) * 32 + 8 * grp + e];
            u32x4 hi, lo;
            split8(x, hi, lo);
            u32x4* f = p.qf + (((int64_t)s * kb_n + kb) * (p.NQ / 16) + row / 16) * 128 + 16 * grp + row % 16;
            f[0] = hi;
            f[64] = lo;
        }
        if (g == 0)      // rows past the query rows
            for (int i = tid; i < (p.NQ - p.rows) * 4; i += 256) {
                const int row = p.rows + (i >> 2), grp = i & 3;
                u32x4* f = p.qf + (((int64_t)s * kb_n + kb) * (p.NQ / 16) + row / 16) * 128 + 16 * grp + row % 16;
                f[0] = f[64] = u32x4{0, 0, 0, 0};
            }
        return;
    }
    const int s = b / p.rows, row = b % p.rows;
    const JSeq& S = p.seq[s];
    const int h = row % p.H, query = row / p.H, g = h / p.hpg;
    const ET* kx = reinterpret_cast<const ET*>(S.kx) + (int64_t)g * p.cap * D;
    const ET* vx = reinterpret_cast<const ET*>(S.vx) + (int64_t)g * p.cap * D;
    const int ne = (int)S.n_exact;
    const int c = tid & 15, eg = tid >> 4;    // 8 dims, exact row group
    float q8[8];
    ld8<F32>(S.q, ((int64_t)query * p.H + h) * D + 8 * c, q8);
    float m = -INFINITY;
    for (int e0 = 0; e0 < ne; e0 += 64) {
        float x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) ld8<F32>(kx, (int64_t)min(e0 + 16 * u + eg, ne - 1) * D + 8 * c, x[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float a = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaf(q8[e], x[u][e], a);
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) a += __shfl_xor(a, o, 64);
            a *= 0.08838834764831845f;
            const int e = e0 + 16 * u + eg;
            if (e < ne) {
                if (c == 0) xs[e] = a;
                m = fmaxf(m, a);
            }
        }
    }
    m = jd_wave_max(m);
    if (lane == 0) wred[0][wave] = m;
    __syncthreads();
    const float M = fmaxf(fmaxf(wred[0][0], wred[0][1]), fmaxf(wred[0][2], wred[0][3]));
    float l = 0.f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    for (int e0 = 0; e0 < ne; e0 += 64) {
        float x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) ld8<F32>(vx, (int64_t)min(e0 + 16 * u + eg, ne - 1) * D + 8 * c, x[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + 16 * u + eg;
            if (e < ne) {
                const float pe = fast_exp(xs[e] - M);
                l += pe;
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] = fmaf(pe, x[u][i], acc[i]);
            }
        }
    }
    l = jd_wave_sum(c == 0 ? l : 0.f);
    if (lane == 0) wred[1][wave] = l;
#pragma unroll
    for (int i = 0; i < 8; ++i) red[eg][8 * c + i] = acc[i];
    __syncthreads();
    float* xr = p.xrec + ((int64_t)s * p.rows + row) * (2 + D);
    if (tid < D) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) a += red[i][tid];
        xr[2 + tid] = a;
    }
    if (tid == 0) { xr[0] = M; xr[1] = ((wred[1][0] + wred[1][1]) + wred[1][2]) + wred[1][3]; }
}

// ---- scores ---------------------------------------------------------------------------------
// A block's coefficients are one contiguous piece of memory: it streams through an LDS ring in
// whole 1 KB direct-to-LDS loads, up to 72 KB ahead (rows loaded straight into MFMA operands
// instead, 64 bytes of 16 unaligned rows per load: 27 us against 18.4 at 32768 tokens, R = 1024;
// each load took 100 cycles to issue).  A wave per slice and tile of 16 tokens, two tiles and one
// barrier per step (8 waves and a tile per step: 20 us).  Operands are 16-byte LDS reads at any
// 2-byte alignment; lanes past their row's end read nothing (18.2 against 20.2 us: LDS is what
// binds, with the vector instructions).  fp32: the ring holds one tile per step (16 rows of 1024
// are 64 KB), so the second eight waves only load; eight waves in all were not measured there.
template <bool F32, int RT> struct JScore {
    static constexpr int NQ = 16 * RT;
    static constexpr int ES = F32 ? 4 : 2;
    static constexpr int TP = F32 ? 1 : 2;                    // tiles per barrier
    static constexpr int RU = F32 ? 96 : 72;                  // ring units of 1 KB; TP tiles take at most 66
    static constexpr int RING = RU * 1024;
    static constexpr int PSUM = RING + 1024;                  // unit 0 again past the end, for reads across it
    static constexpr int SC = PSUM + 2 * 8 * TP * 16 * NQ * 4;   // [2][slice][16 TP][NQ]
    static constexpr size_t LDS = SC + JS_B * NQ * 4;         // [128][NQ] the block's scores
};

template <bool F32, int RT>
__global__ __launch_bounds__(JS_T, 4) void js_kernel(JDec p) {
    typedef JScore<F32, RT> C;
    constexpr int NQ = C::NQ, QC = NQ / 4;         // 16-byte chunks of a token's scores
    constexpr uint32_t ES = C::ES, RING = C::RING;
    constexpr int TT = 16 * C::TP;                 // tokens per barrier
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float* psum = reinterpret_cast<float*>(smem + C::PSUM);
    float* sc_b = reinterpret_cast<float*>(smem + C::SC);
    __shared__ uint32_t so[JS_B + 1];              // first byte of token i's row, from the block's first 16 bytes
    __shared__ uint32_t sw[JS_B];                  // the same within the ring
    __shared__ float red[2][JS_T / 64][NQ];
    const int s = blockIdx.x / p.s_wg, x = blockIdx.x % p.s_wg;
    const JSeq& S = p.seq[s];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nsl = p.R / JSL;
    const int slice = wave & 7, tp = wave >> 3;
    const bool mine = slice < nsl && tp < C::TP;   // the other waves only load
    const uint32_t ring0 = lds_addr(smem);
    // q' of this wave's slice: lane -> row 16 rt + l16, coefficients 128 slice + 32 st + 8 grp ..
    u32x4 qf[RT][4][2];
    {
        const u32x4* f = p.qf + ((int64_t)s * nsl + (mine ? slice : 0)) * 4 * RT * 128 + lane;
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int h = 0; h < 2; ++h) qf[rt][st][h] = f[((st * RT + rt) * 2 + h) * 64];
    }
    for (int blk = x; blk < p.n_blk; blk += p.s_wg) {
        const int64_t t0 = (int64_t)blk * p.bt;
        const int T = (int)min((int64_t)p.bt, p.N - t0);
        const uint64_t first = (uint64_t)S.offset[t0] * ES & ~15ull, last = (uint64_t)S.offset[t0 + T] * ES;
        if (tid <= JS_B) {
            const uint32_t o = (uint32_t)((uint64_t)S.offset[t0 + min(tid, T)] * ES - first);
            so[tid] = o;
            if (tid < JS_B) sw[tid] = o % RING;
        }
        __syncthreads();
        // ---- the ring: unit u (1 KB from first + 1024 u) by wave u % 16 into slot u % RU
        const uint8_t* src = (const uint8_t*)S.coef + first;
        const uint32_t bytes = (uint32_t)(last - first);
        const int units = __builtin_amdgcn_readfirstlane((int)((bytes + 1023) >> 10));
        const uint32_t end16 = bytes ? (bytes - 1) & ~15u : 0;
        int iu = wave, slot = wave;                // this wave's next unit and its slot
        auto issue = [&](int to) {                 // own units before `to`
            for (; iu < to; iu += 16) {
                const uint8_t* a = src + min((uint32_t)iu * 1024u + 16u * lane, end16);
                gemm_load(a, ring0 + 1024u * (uint32_t)slot);
                if (slot == 0) gemm_load(a, ring0 + RING);
                slot += 16;
                if (slot >= C::RU) slot -= C::RU;
            }
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int lim = min(units, C::RU);               // every wave's units before lim are issued
        issue(lim);
        auto reduce = [&](int t) {                 // the partial scores of group t, the slices in order
#pragma unroll
            for (int i = 0; i < (TT * NQ + JS_T - 1) / JS_T; ++i) {
                const int tk = (tid + JS_T * i) / NQ, q = tid % NQ;
                if (tk < TT) {
                    const float* ps = psum + (t & 1) * 8 * TT * NQ + tk * NQ + (((q >> 2) ^ (tk & (QC - 1))) << 2) + (q & 3);
                    float v = ps[0];
#pragma unroll
                    for (int c = 1; c < 8; ++c)
                        if (c < nsl) v += ps[c * TT * NQ];
                    sc_b[(TT * t + tk) * NQ + q] = v;
                }
            }
        };
        const int groups = (T + TT - 1) / TT;
        for (int t = 0; t < groups; ++t) {
            const uint32_t us = __builtin_amdgcn_readfirstlane(so[TT * t]) >> 10;
            const int ue = (int)((__builtin_amdgcn_readfirstlane(so[TT * t + TT]) + 1023) >> 10);
            if (lim < ue) {                        // group t did not fit behind the one before it
                __syncthreads();                   // which now is done
                issue(lim = min(units, (int)us + C::RU));
            }
            jd_wait(iu > ue ? (iu - ue) / 16 : 0);  // own units from ue on may be in flight
            __syncthreads();                       // group t has landed, groups before t are done
            issue(lim = min(units, (int)us + C::RU));
            if (mine) {
                {
                    const int tok = TT * t + 16 * tp + l16;
                    const int r = (int)min((so[tok + 1] - so[tok]) / ES, (uint32_t)p.R);
                    const int nv = r - slice * JSL - 8 * grp;
                    const uint32_t at = sw[tok] + (uint32_t)(slice * JSL + 8 * grp) * ES;
                    f32x4 sc[RT][2];               // hi and lo parts of q'
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) sc[rt][0] = sc[rt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                    const bool part = __any(nv < 128 - 8 * grp);   // a row ends in this slice
                    if (__any(nv > 0)) {
#pragma unroll
                        for (int st = 0; st < 4; ++st) {
                            const uint32_t a = min(at + 32 * st * ES, at + 32 * st * ES - RING);     // within the ring
                            const int nk = min(max(nv - 32 * st, 0), 8);
                            u32x4 kh, kl;
                            if constexpr (F32) {
                                const float* w = reinterpret_cast<const float*>(smem + a);
                                float x8[8];
#pragma unroll
                                for (int e = 0; e < 8; ++e) { const float v = w[e]; x8[e] = e < nk ? v : 0.f; }
                                split8(x8, kh, kl);
                            } else {
                                // lanes past their row's end read nothing: fewer banks to serve
                                kh = u32x4{0u, 0u, 0u, 0u};
                                if (nk > 0) __builtin_memcpy(&kh, smem + a, 16);   // any 2-byte alignment
                                if (part) kh = keep_first(kh, nk);
                            }
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) {
                                sc[rt][0] = mfma(qf[rt][st][0], kh, sc[rt][0]);
                                sc[rt][1] = mfma(qf[rt][st][1], kh, sc[rt][1]);
                                if constexpr (F32) sc[rt][1] = mfma(qf[rt][st][0], kl, sc[rt][1]);
                            }
                        }
                    }
                    const int row = 16 * tp + l16;
                    f32x4* ps = reinterpret_cast<f32x4*>(psum) + (((t & 1) * 8 + slice) * TT + row) * QC;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) ps[(4 * rt + grp) ^ (row & (QC - 1))] = sc[rt][0] + sc[rt][1];
                }
            }
            if (t > 0) reduce(t - 1);
        }
        __syncthreads();
        reduce(groups - 1);
        __syncthreads();
        // ---- the block's scores out, their maximum and sum of exponentials per row
        const int tk = tid / NQ, q = tid % NQ;     // tokens tk, tk + JS_T / NQ, ..
        constexpr int TS = JS_T / NQ, PPT = JS_B / TS;
        float* So = p.S + ((int64_t)s * p.n_blk * p.bt + t0) * NQ;
        float v[PPT], m = -INFINITY, l = 0.f;
#pragma unroll
        for (int i = 0; i < PPT; ++i) {
            const bool ok = tk + TS * i < T;
            v[i] = ok ? sc_b[(tk + TS * i) * NQ + q] : -INFINITY;
            if (ok) So[(tk + TS * i) * NQ + q] = v[i];
            m = fmaxf(m, v[i]);
        }
#pragma unroll
        for (int o = NQ; o < 64; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if (lane < NQ) red[0][wave][q] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < JS_T / 64; ++w) m = fmaxf(m, red[0][w][q]);
#pragma unroll
        for (int i = 0; i < PPT; ++i) l += tk + TS * i < T ? fast_exp(v[i] - m) : 0.f;
#pragma unroll
        for (int o = NQ; o < 64; o <<= 1) l += __shfl_xor(l, o, 64);
        if (lane < NQ) red[1][wave][q] = l;
        __syncthreads();
        if (tid < NQ) {
            l = red[1][0][q];
#pragma unroll
            for (int w = 1; w < JS_T / 64; ++w) l += red[1][w][q];
            float* ml = p.ml + ((int64_t)s * p.n_blk + blk) * 2 * NQ;
            ml[q] = m;
            ml[NQ + q] = l;
        }
    }
}

// ---- values ---------------------------------------------------------------------------------
// Rounds of E rows (a row: up to 128 coefficients of one token), the next one's loads in flight
// during a round's products.  LDS: the rows (bf16; fp32: hi and lo planes), shifted and cut on the
// way, and their softmax weights [row][NQ] as hi and lo parts, both read transposed
// (ds_read_b64_tr_b16: 4 rows x 16 columns per 16 lanes).  Row strides leave the 8 rows x 32 bytes
// that half a wave reads in all 64 banks.  Bound by instructions: rows kept as they lie in memory
// and gathered by element (4 reads where one transposed read does) 23 us, a wave per 64 tokens
// from lists to products 23 us, against 19 (32768 tokens, R = 1024).
template <bool F32, int RT> struct JVal {
    static constexpr int NQ = 16 * RT;
    static constexpr int E = F32 ? 128 : 256;
    static constexpr int CS = 288, PS = RT == 2 ? 96 : 32;          // row strides, bytes
    static constexpr int PLANES = F32 ? 2 : 1;
    static constexpr int LMAX = 2 * (JV_B + 32);                    // rows of a block's two lists
    static constexpr size_t LDS = (size_t)PLANES * E * CS + 2 * (size_t)E * PS + (size_t)LMAX * 8;
};

typedef short jv_s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 tr_read(const jd_lds* p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) jv_s16x4*)p));
}

template <bool F32, int RT>
__global__ __launch_bounds__(JV_T, 4) void jv_kernel(JDec p) {
    typedef JVal<F32, RT> C;
    constexpr int NQ = C::NQ, E = C::E;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint8_t* cbuf = smem;
    uint8_t* pbuf = smem + C::PLANES * E * C::CS;
    uint32_t* l_off = reinterpret_cast<uint32_t*>(pbuf + 2 * E * C::PS);           // row's first coefficient
    uint16_t* l_nv = reinterpret_cast<uint16_t*>(l_off + C::LMAX);                 // coefficients (0: padding)
    uint16_t* l_tok = l_nv + C::LMAX;                                              // token of the block
    __shared__ int wc[2][JV_B / 64];
    __shared__ float red[JV_T / NQ][NQ];
    __shared__ float Mrow[NQ];
    const int np = p.R / JSL / 2;                 // slice pairs
    const int per = p.n_sp * np;
    const int s = blockIdx.x / per, lb = blockIdx.x % per;
    // the pairs of a range share memory lines: workgroup L runs on XCD L mod 8, keep them on one
    int sp, pair;
    if (p.n_sp % 8 == 0) { sp = lb / (8 * np) * 8 + lb % 8; pair = lb / 8 % np; }
    else { sp = lb / np; pair = lb % np; }
    const int sl[2] = {pair, 2 * np - 1 - pair};
    const JSeq& S = p.seq[s];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int cw = wave & 7, half = wave >> 3;    // coordinates 16 cw .. + 15; steps of this parity
    const int64_t t0 = (int64_t)sp * p.tps, t1 = min(t0 + p.tps, p.N);
    const float* Sc = p.S + (int64_t)s * p.n_blk * p.bt * NQ;
    uint32_t o0 = 0, o1 = 0;
    auto meta = [&](int64_t tb) {
        const int64_t t = tid < JV_B ? min(tb + tid, t1) : t1;
        o0 = S.offset[t];
        o1 = S.offset[min(t + 1, t1)];
    };
    meta(t0);
    // ---- the frame: every block's maximum
    {
        const int row = tid % NQ, g0 = tid / NQ;
        const float* ml = p.ml + (int64_t)s * p.n_blk * 2 * NQ + row;
        float m = -INFINITY;
#pragma unroll 16
        for (int b = g0; b < p.n_blk; b += JV_T / NQ) m = fmaxf(m, ml[(int64_t)b * 2 * NQ]);
        red[g0][row] = m;
    }
    f32x4 acc[2][RT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[a][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t tb = t0; tb < t1; tb += JV_B) {
        // ---- the two slices' rows of this block, each list padded to 32
        const int r = (int)min(o1 - o0, (uint32_t)p.R);
        int pos[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const uint64_t m = __ballot(r > sl[a] * JSL);
            pos[a] = __popcll(m & ((1ull << lane) - 1));
            if (lane == 0 && wave < JV_B / 64) wc[a][wave] = __popcll(m);
        }
        __syncthreads();                          // also: the last round's rows have been read
        int tot[2] = {0, 0};
#pragma unroll
        for (int w = 0; w < JV_B / 64; ++w)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                pos[a] += w < wave ? wc[a][w] : 0;
                tot[a] += wc[a][w];
            }
        const int pad0 = (tot[0] + 31) & ~31, pad1 = (tot[1] + 31) & ~31, n_rows = pad0 + pad1;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (r > sl[a] * JSL) {
                const int at = (a ? pad0 : 0) + pos[a];
                l_off[at] = o0 + (uint32_t)(sl[a] * JSL);
                l_nv[at] = (uint16_t)min(r - sl[a] * JSL, JSL);
                l_tok[at] = (uint16_t)tid;
            }
            if (tid < (a ? pad1 - tot[1] : pad0 - tot[0])) {
                const int at = (a ? pad0 : 0) + tot[a] + tid;
                l_off[at] = 0;
                l_nv[at] = 0;
                l_tok[at] = 0;
            }
        }
        if (tid < NQ) {
            float m = red[0][tid];
#pragma unroll
            for (int i = 1; i < JV_T / NQ; ++i) m = fmaxf(m, red[i][tid]);
            Mrow[tid] = m;
        }
        __syncthreads();
        // ---- rounds of E rows, the next one's loads in flight during the products
        constexpr int NI = E * 16 / JV_T;         // row pieces of 8 coefficients per thread
        constexpr int QC = NQ / 4, SI = (E * QC + JV_T - 1) / JV_T;   // 4 weights per thread and pass
        Raw8<F32> cf[NI];
        f32x4 sc[SI];
        auto fetch = [&](int e0) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int e = min(e0 + (tid >> 4) + (JV_T / 16) * i, n_rows - 1);
                cf[i] = ld_raw8<F32>(S.coef, l_off[e] + (8 * (tid & 15) < (int)l_nv[e] ? 8u * (tid & 15) : 0u));
            }
#pragma unroll
            for (int i = 0; i < SI; ++i) {
                const int e = min(e0 + (tid + JV_T * i) / QC, n_rows - 1);
                sc[i] = ld4(Sc + (tb + l_tok[e]) * NQ + 4 * (tid % QC));
            }
        };
        if (n_rows > 0) fetch(0);
        if (tb + JV_B < t1) meta(tb + JV_B);
        for (int e0 = 0; e0 < n_rows; e0 += E) {
            if (e0) __syncthreads();              // the last round's rows have been read
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int e = (tid >> 4) + (JV_T / 16) * i, ee = e0 + e;
                u32x4 hi, lo;
                frag8<F32>(cf[i], ee < n_rows ? min(max((int)l_nv[min(ee, n_rows - 1)] - 8 * (tid & 15), 0), 8) : 0, hi, lo);
                *reinterpret_cast<u32x4*>(cbuf + e * C::CS + 16 * (tid & 15)) = hi;
                if constexpr (F32) *reinterpret_cast<u32x4*>(cbuf + (E + e) * C::CS + 16 * (tid & 15)) = lo;
            }
#pragma unroll
            for (int i = 0; i < SI; ++i) {
                const int e = (tid + JV_T * i) / QC, f0 = 4 * (tid % QC);
                const bool ok = e0 + e < n_rows && l_nv[min(e0 + e, n_rows - 1)] != 0;
                float w[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) w[v] = ok ? fast_exp(sc[i][v] - Mrow[f0 + v]) : 0.f;
                uint2 hi, lo;
                split2(w[0], w[1], hi.x, lo.x);
                split2(w[2], w[3], hi.y, lo.y);
                if (e < E) {
                    *reinterpret_cast<uint2*>(pbuf + e * C::PS + 2 * f0) = hi;
                    *reinterpret_cast<uint2*>(pbuf + (E + e) * C::PS + 2 * f0) = lo;
                }
            }
            __syncthreads();
            if (e0 + E < n_rows) fetch(e0 + E);
            // A: coordinates 16 cw + l16 x 32 rows; B: the same rows x 16 query rows
            const jd_lds* ca = (const jd_lds*)cbuf + (4 * grp + (l16 >> 2)) * C::CS + 32 * cw + 8 * (l16 & 3);
            const jd_lds* pa = (const jd_lds*)pbuf + (4 * grp + (l16 >> 2)) * C::PS + 8 * (l16 & 3);
            auto step = [&](int k, f32x4 (&ac)[RT]) {
                u32x4 a[C::PLANES];
#pragma unroll
                for (int h = 0; h < C::PLANES; ++h) {
                    const uint2 u = tr_read(ca + (h * E + 32 * k) * C::CS), v = tr_read(ca + (h * E + 32 * k + 16) * C::CS);
                    a[h] = u32x4{u.x, u.y, v.x, v.y};
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    u32x4 b[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint2 u = tr_read(pa + (h * E + 32 * k) * C::PS + 32 * rt);
                        const uint2 v = tr_read(pa + (h * E + 32 * k + 16) * C::PS + 32 * rt);
                        b[h] = u32x4{u.x, u.y, v.x, v.y};
                    }
                    ac[rt] = mfma(a[0], b[0], ac[rt]);
                    ac[rt] = mfma(a[0], b[1], ac[rt]);
                    if constexpr (F32) ac[rt] = mfma(a[1], b[0], ac[rt]);
                }
            };
            const int k1 = min(E, n_rows - e0) / 32, k0 = min(max(pad0 - e0, 0) / 32, k1);
#pragma unroll 2
            for (int k = half; k < k0; k += 2) step(k, acc[0]);
#pragma unroll 2
            for (int k = k0 + ((k0 ^ half) & 1); k < k1; k += 2) step(k, acc[1]);
        }
    }
    // ---- the two halves' sums added
    __syncthreads();
    f32x4* sums = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
            if (half) sums[((cw * 2 + a) * RT + rt) * 64 + lane] = acc[a][rt];
    __syncthreads();
    if (half) return;
    float* rec = p.rec + ((int64_t)s * p.n_sp + sp) * NQ * p.R;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
            *reinterpret_cast<f32x4*>(rec + (int64_t)(16 * rt + l16) * p.R + sl[a] * JSL + 16 * cw + 4 * grp) =
                acc[a][rt] + sums[((cw * 2 + a) * RT + rt) * 64 + lane];
}

// ---- rotation back --------------------------------------------------------------------------
// part[s][g][kb][r][i] = sum over 32 coefficients k of W_V,g[k][i] (sum over the ranges of rec);
// latency: the basis entries and a thread's records all in flight
__global__ __launch_bounds__(256) void jc_kernel(JDec p) {
    __shared__ __attribute__((aligned(16))) f32x4 red[256];
    __shared__ __attribute__((aligned(16))) float comb[JROWS][JC_K];
    __shared__ float half[JROWS][D];
    const int kb_n = p.R / JC_K;
    const int s = blockIdx.x / (p.G * kb_n), g = blockIdx.x / kb_n % p.G, kb = blockIdx.x % kb_n;
    const int tid = threadIdx.x, i = tid & 127, kh = tid >> 7;
    const int Dz = 2 * p.G * D, k0 = kb * JC_K;
    const float* w = p.W + (int64_t)(k0 + 16 * kh) * Dz + (p.G + g) * D + i;
    float wv[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) wv[m] = w[(int64_t)m * Dz];
    const int items = p.nr * 8, ng = 256 / items;     // (row, 4 coefficients), thread groups over the ranges
    const int it = tid % items, xg = tid / items;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
    if (xg < ng) {
        const int r = it >> 3;
        const float* src = p.rec + ((int64_t)s * p.n_sp * p.NQ + (r / p.hpg) * p.H + g * p.hpg + r % p.hpg) * p.R + k0 + 4 * (it & 7);
#pragma unroll 8
        for (int x = xg; x < p.n_sp; x += ng) a = a + ld4(src + (int64_t)x * p.NQ * p.R);
    }
    red[tid] = a;
    __syncthreads();
    if (tid < items) {
        for (int x = 1; x < ng; ++x) a = a + red[x * items + tid];
        *reinterpret_cast<f32x4*>(&comb[tid >> 3][4 * (tid & 7)]) = a;
    }
    __syncthreads();
    float* dst = p.part + (((int64_t)s * p.G + g) * kb_n + kb) * p.nr * D + i;
    if (kh) {
        for (int r = 0; r < p.nr; ++r) {
            float v = 0.f;
#pragma unroll
            for (int m = 0; m < 16; ++m) v = fmaf(wv[m], comb[r][16 + m], v);
            half[r][i] = v;
        }
    }
    __syncthreads();
    if (!kh) {
        for (int r = 0; r < p.nr; ++r) {
            float v = 0.f;
#pragma unroll
            for (int m = 0; m < 16; ++m) v = fmaf(wv[m], comb[r][m], v);
            dst[r * D] = v + half[r][i];
        }
    }
}

// out = (parts in the frame M + exp(m_x - M) acc_x) / L per query row
template <bool F32>
__global__ __launch_bounds__(256) void jo_kernel(JDec p) {
    typedef typename std::conditional<F32, float, uint16_t>::type ET;
    __shared__ float wm[4], wl[4], half[D];
    const int s = blockIdx.x / p.rows, row = blockIdx.x % p.rows;
    const int h = row % p.H, query = row / p.H, g = h / p.hpg;
    const int r = query * p.hpg + h % p.hpg;      // the row's index among head g's rows
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = tid & 127, kh = tid >> 7;
    const int kb_n = p.R / JC_K;
    const float* src = p.part + ((int64_t)s * p.G + g) * kb_n * p.nr * D + r * D + i;
    const float* xr = p.xrec + ((int64_t)s * p.rows + row) * (2 + D);
    const float xm = xr[0], xl = xr[1], xa = xr[2 + i];
    float a = 0.f;
#pragma unroll 16
    for (int x = kh; x < kb_n; x += 2) a += src[(int64_t)x * p.nr * D];
    const float* ml = p.ml + (int64_t)s * p.n_blk * 2 * p.NQ + row;
    float m = -INFINITY, l = 0.f;
    for (int b = tid; b < p.n_blk; b += 256) {
        const float mb = ml[(int64_t)b * 2 * p.NQ], lb = ml[((int64_t)b * 2 + 1) * p.NQ];
        const float mn = fmaxf(m, mb);
        l = (m == -INFINITY ? 0.f : l * fast_exp(m - mn)) + lb * fast_exp(mb - mn);
        m = mn;
    }
    const float mw = jd_wave_max(m);
    if (lane == 0) wm[wave] = mw;
    if (kh) half[i] = a;
    __syncthreads();
    const float Mc = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));   // the frame of the parts
    l = jd_wave_sum(m == -INFINITY ? 0.f : l * fast_exp(m - Mc));
    if (lane == 0) wl[wave] = l;
    __syncthreads();
    if (kh) return;
    const float M = fmaxf(Mc, xm), fc = fast_exp(Mc - M), fx = fast_exp(xm - M);
    const float L = (((wl[0] + wl[1]) + wl[2]) + wl[3]) * fc + xl * fx;
    ET* out = reinterpret_cast<ET*>(p.seq[s].out) + ((int64_t)query * p.H + h) * D;
    out[i] = to_elem<ET>(((a + half[i]) * fc + fx * xa) / L);
}

struct JPlan { int NQ, bt, n_blk, s_wg, n_sp, tps; size_t qp, S, ml, rec, xrec, part; };

// per launch: about one workgroup per CU for the scores and for the values, but no range of fewer
// than 64 tokens (a range leaves a record of NQ x R sums)
static JPlan joint_plan(const varrate_shape& sh, int R, int S, int rows) {
    JPlan pl;
    const int64_t N = sh.n - sh.w;
    const int ns = S < JSEQ ? S : JSEQ, np = R / JSL / 2;
    pl.NQ = rows > 16 ? 32 : 16;
    // a block's time is that of its steps in turn (1.4 us each), so few tokens go in smaller blocks
    pl.bt = JS_B;
    while (pl.bt > 32 && ns * ((N + pl.bt - 1) / pl.bt) < 128) pl.bt /= 2;
    pl.n_blk = (int)((N + pl.bt - 1) / pl.bt);
    pl.s_wg = 256 / ns < pl.n_blk ? 256 / ns : pl.n_blk;
    int64_t sp = 256 / (ns * np);
    if (sp > (N + 63) / 64) sp = (N + 63) / 64;
    if (sp < 1) sp = 1;
    pl.tps = (int)(((N + sp - 1) / sp + 31) / 32 * 32);
    pl.n_sp = (int)((N + pl.tps - 1) / pl.tps);
    pl.qp = align256((size_t)S * pl.NQ * R * 4);
    pl.S = align256((size_t)S * pl.n_blk * pl.bt * pl.NQ * 4);
    pl.ml = align256((size_t)S * pl.n_blk * 2 * pl.NQ * 4);
    pl.rec = align256((size_t)S * pl.n_sp * pl.NQ * R * 4);
    pl.xrec = align256((size_t)S * rows * (2 + D) * 4);
    pl.part = align256((size_t)S * rows * (R / JC_K) * D * 4);   // G heads of rows / G rows
    return pl;
}

size_t joint_decode_ws_bytes(const varrate_shape& sh, int R, int S, int Q) {
    const JPlan pl = joint_plan(sh, R, S, Q * sh.H);
    return pl.qp + pl.S + pl.ml + pl.rec + pl.xrec + pl.part;
}

template <bool F32, int RT>
static hipError_t launch_group(const JDec& p, hipStream_t st) {
    typedef JVal<F32, RT> C;
    const size_t s_lds = JScore<F32, RT>::LDS;
    const unsigned np = (unsigned)(p.R / JSL / 2);
    hipError_t e = ensure_lds_limit((const void*)js_kernel<F32, RT>, s_lds);
    if (e != hipSuccess) return e;
    if ((e = ensure_lds_limit((const void*)jv_kernel<F32, RT>, C::LDS)) != hipSuccess) return e;
    jq_kernel<F32><<<(unsigned)(p.ns * (p.rows + p.G * (p.R / 32))), 256, 0, st>>>(p);
    js_kernel<F32, RT><<<(unsigned)(p.ns * p.s_wg), JS_T, s_lds, st>>>(p);
    jv_kernel<F32, RT><<<(unsigned)p.ns * p.n_sp * np, JV_T, C::LDS, st>>>(p);
    jc_kernel<<<(unsigned)(p.ns * p.G * (p.R / JC_K)), 256, 0, st>>>(p);
    jo_kernel<F32><<<(unsigned)(p.ns * p.rows), 256, 0, st>>>(p);
    return hipGetLastError();
}

hipError_t launch_joint_decode(const varrate_shape& sh, int R, const varrate_jcache* caches, int S, const void* q,
                               int Q, const float* W, void* out, uint8_t* ws, hipStream_t st) {
    const int rows = Q * sh.H;
    if (rows > JROWS) return hipErrorInvalidValue;
    const JPlan pl = joint_plan(sh, R, S, rows);
    const bool f32 = sh.dtype != VARRATE_BF16;
    const size_t qstride = (size_t)Q * sh.H * D * (f32 ? 4 : 2);
    for (int s0 = 0; s0 < S; s0 += JSEQ) {
        JDec p;
        p.ns = S - s0 < JSEQ ? S - s0 : JSEQ;
        for (int i = 0; i < JSEQ; ++i) {
            const int si = s0 + (i < p.ns ? i : 0);
            const varrate_jcache& c = caches[si];
            p.seq[i] = JSeq{c.coef, c.offset, c.k_exact, c.v_exact, (const uint8_t*)q + si * qstride,
                            (uint8_t*)out + si * qstride, c.n_exact};
        }
        p.W = W;
        p.N = sh.n - sh.w;
        p.cap = caches[s0].cap;
        p.G = sh.G;
        p.H = sh.H;
        p.hpg = sh.H / sh.G;
        p.rows = rows;
        p.nr = rows / sh.G;
        p.NQ = pl.NQ;
        p.R = R;
        p.bt = pl.bt;
        p.n_blk = pl.n_blk;
        p.s_wg = pl.s_wg;
        p.n_sp = pl.n_sp;
        p.tps = pl.tps;
        uint8_t* b = ws;
        p.qf = (u32x4*)b + (size_t)s0 * pl.NQ * R / 4;                     b += pl.qp;
        p.S = (float*)b + (size_t)s0 * pl.n_blk * pl.bt * pl.NQ;           b += pl.S;
        p.ml = (float*)b + (size_t)s0 * pl.n_blk * 2 * pl.NQ;             b += pl.ml;
        p.rec = (float*)b + (size_t)s0 * pl.n_sp * pl.NQ * R;             b += pl.rec;
        p.xrec = (float*)b + (size_t)s0 * rows * (2 + D);                 b += pl.xrec;
        p.part = (float*)b + (size_t)s0 * rows * (R / JC_K) * D;
        const hipError_t e = f32 ? (rows > 16 ? launch_group<true, 2>(p, st) : launch_group<true, 1>(p, st))
                                 : (rows > 16 ? launch_group<false, 2>(p, st) : launch_group<false, 1>(p, st));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace vr
