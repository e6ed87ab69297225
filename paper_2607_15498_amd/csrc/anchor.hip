// Residual codec with strided anchors (Sec. 3.1 "Residual codec", Eq. (2); Algorithm 1):
// compress-side kernels, gfx950.
//
// Anchors are the prefix tokens t = a delta (a = 0 .. na - 1, t < N); they and the window
// stay exact.  Coded token number i (the prefix tokens that are not anchors, in order) is
// token t(i) = i + i / (delta - 1) + 1.  Each coded token is coded as its residual to the mean
// of its c = 4 nearest anchors in Euclidean distance over the joint vector
// z_t = [k_t of all heads; v_t of all heads] (2 G d elements).
//
//   anc_norms    ||z_a||^2 of every anchor (fp32, fixed summation order)
//   anc_search   distance GEMM <z_a, z_t> by bf16 MFMA (the bf16 inputs are exact, the fp32
//                accumulation is the only rounding) on tiles of 256 x 256 or 128 anchors x 64
//                tokens; ranking key ||z_a||^2 - 2 <z_a, z_t> (||z_t||^2 is common to a
//                token's candidates); each tile leaves every token's 4 best (key, anchor) pairs
//   anc_merge    a token's partial lists -> its 4 nearest anchors, nearest first (ties to the
//                lower anchor number)
//   anc_prep     coded salience gathered from the prefix's, residuals k_t - mean, v_t - mean
//                (fp32, stored in the layer's dtype) followed by the window rows, and the
//                anchor rows copied to their store
//   anc_count, anc_lists, anc_fill  after the allocation: the anchors of each stored position,
//                per anchor the stored positions that use it (counts, scan, fill), and those
//                lists cut into pieces of 64 entries (hub anchors are used by most tokens)
#include "vr_gemm.h"
#include "vr_internal.h"

namespace vr {

constexpr int AN_C = 4;                 // nearest anchors per coded token
constexpr int AN_TA = 128;              // anchors per search tile at least (32 CF)

// A token's four anchor numbers in the caller's lists, which are 2-byte aligned.
__device__ __forceinline__ uint2 anc_near(const uint16_t* p) {
    uint2 v;
    __builtin_memcpy(&v, p, 8);
    return v;
}
__device__ __forceinline__ void anc_near_out(uint16_t* p, uint2 v) { __builtin_memcpy(p, &v, 8); }

__host__ __device__ inline int64_t anc_token(int64_t i, int delta) { return i + i / (delta - 1) + 1; }

// ---- anchor norms: one wave per anchor, its row staged in LDS by 16-byte loads and summed
// with lane l taking elements l, l + 64, .. in order (latency bound: 14 us for 2046 anchors of
// 2048 elements with 2-byte loads, 4.8 with these)
constexpr int AN_NP = 2048;             // elements staged at a time
__global__ __launch_bounds__(256) void anc_norms(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                                                int64_t na, int delta, int GD, float* __restrict__ nrm) {
    __shared__ __attribute__((aligned(16))) uint16_t row[4][AN_NP];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t a = (int64_t)blockIdx.x * 4 + wave;
    if (a >= na) return;                // (no workgroup barrier below)
    const int64_t t = a * delta;
    float s = 0.f;
    for (int k0 = 0; k0 < 2 * GD; k0 += AN_NP) {
        const int n = 2 * GD - k0 < AN_NP ? 2 * GD - k0 : AN_NP;        // a multiple of 256
        u32x4 w[AN_NP / 512];
#pragma unroll
        for (int u = 0; u < AN_NP / 512; ++u) {
            const int e = 512 * u + 8 * lane, k = k0 + (e < n ? e : 0);
            w[u] = load16(k < GD ? K + t * GD + k : V + t * GD + k - GD);
        }
#pragma unroll
        for (int u = 0; u < AN_NP / 512; ++u) *reinterpret_cast<u32x4*>(&row[wave][512 * u + 8 * lane]) = w[u];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 8
        for (int k = lane; k < n; k += 64) {
            const float x = bf16_to_f32(row[wave][k]);
            s = fmaf(x, x, s);
        }
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) nrm[a] = s;
}

// The 4 best (smallest key, ties to the smaller anchor number), sorted, as fp64 values whose
// high words are the fp32 keys and whose low words are the anchor numbers (complemented under
// a negative key): doubles order by sign, then by the remaining 63 bits, so they order as
// (key, anchor) pairs do and a compare-exchange is one minimum and one maximum.  An fp32
// infinity is a finite double there; NaN keys come behind it, whatever their payload, and the
// largest pattern used, AN_NONE, stands for no anchor.
typedef double Top4[AN_C];
constexpr uint32_t AN_NAN = 0x7F800001u;                          // high word of a NaN key
constexpr unsigned long long AN_NONE = ((unsigned long long)AN_NAN << 32) | 0xFFFFFFFFull;
__device__ __forceinline__ double anc_pack(float key, uint32_t a) {
    const uint32_t k = key == key ? __float_as_uint(key) : AN_NAN;
    const uint32_t lo = a ^ (uint32_t)((int32_t)k >> 31);
    return __builtin_bit_cast(double, ((unsigned long long)k << 32) | lo);
}
__device__ __forceinline__ uint32_t anc_number(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    return (uint32_t)b ^ (uint32_t)((int64_t)b >> 63);
}
__device__ __forceinline__ double anc_min(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double anc_max(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ void anc_cx(double& a, double& b) {
    const double t = anc_min(a, b);
    b = anc_max(a, b);
    a = t;
}
__device__ __forceinline__ void top4_sort(Top4& t) {
    anc_cx(t[0], t[1]);
    anc_cx(t[2], t[3]);
    anc_cx(t[0], t[2]);
    anc_cx(t[1], t[3]);
    anc_cx(t[1], t[2]);
}
// t = the 4 smallest of two sorted lists, sorted (a bitonic half-cleaner, then its merge)
__device__ __forceinline__ void top4_merge(Top4& t, const Top4& o) {
#pragma unroll
    for (int q = 0; q < AN_C; ++q) t[q] = anc_min(t[q], o[AN_C - 1 - q]);
    anc_cx(t[0], t[2]);
    anc_cx(t[1], t[3]);
    anc_cx(t[0], t[1]);
    anc_cx(t[2], t[3]);
}
// merged with the list of lane ^ 16 (SWAP 16) or lane ^ 32
template <int SWAP> __device__ __forceinline__ void top4_lanes(Top4& t) {
    Top4 o;
    const bool upper = (threadIdx.x & SWAP) != 0;
#pragma unroll
    for (int q = 0; q < AN_C; ++q) {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, t[q]);
        uint32_t w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t x = (uint32_t)(b >> (32 * h));
            // of the two results one is the lane's own value and the other its partner's
            if constexpr (SWAP == 16) {
                const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
                w[h] = upper ? r[0] : r[1];
            } else {
                const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
                w[h] = upper ? r[0] : r[1];
            }
        }
        o[q] = __builtin_bit_cast(double, ((unsigned long long)w[1] << 32) | w[0]);
    }
    top4_merge(t, o);
}

// ---- distance products and each anchor tile's 4 best per token: a workgroup per (64 TF tokens,
// 32 CF anchors), gemm_tile with the anchors as columns.  C[anchor][token]: lane -> token
// column (lane % 16) and anchors 4 (lane / 16) + v of each 16-anchor tile, so a lane sorts 16
// keys per token in registers, the four lanes of a token merge by lane swaps, the two anchor
// halves through LDS.  Workgroups are mapped so that an XCD takes consecutive token tiles of one
// anchor tile, whose rows (1 MB) stay in its L2.  Matrix-core bound; 32768-token Llama layer
// (2046 anchors, 257 GFLOP): 508 us with 64 x 64 wave tiles and lists kept by insertion, 252 us
// now (1020 TFLOP/s).  Ordering NaN keys behind infinite ones is 1.5 us of it (whole compressions,
// 428.0 -> 429.5); taking them for infinite, with a second look only where a wave has fewer than
// four finite keys, costs the same.
struct AnSearch {
    const uint16_t* K;
    const uint16_t* V;
    const float* nrm;
    double* part;       // [n_atiles][Nc][4] packed partial lists
    int64_t Nc, na;
    int delta, GD, n_ttiles, n_atiles;
};

template <int TF, int CF>
__global__ __launch_bounds__(512, 2) void anc_search(AnSearch p) {
    typedef GemmTile<TF, CF, false> T;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int col = lane & 15, grp = lane >> 4;
    const int wa = wave >> 2, wt = wave & 3;
    // XCD x (workgroup id mod 8) takes the x-th eighth of the anchor-tile-major order
    const int per = (p.n_ttiles * p.n_atiles + 7) / 8, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const int at = id / p.n_ttiles, tt = id % p.n_ttiles;
    if (at >= p.n_atiles) return;
    const int64_t i0 = (int64_t)tt * T::TOK;
    const int64_t a0 = (int64_t)at * T::ROWS;
    // rows past the anchors or tokens are clamped here and dropped later
    const uint8_t* tok[T::TL];
#pragma unroll
    for (int u = 0; u < T::TL; ++u) {
        int64_t i = i0 + gemm_row(T::TL * wave + u);
        i = i < p.Nc ? i : p.Nc - 1;
        tok[u] = reinterpret_cast<const uint8_t*>(p.K + anc_token(i, p.delta) * p.GD + 8 * gemm_piece());
    }
    const uint8_t* anc[T::CL];
#pragma unroll
    for (int u = 0; u < T::CL; ++u) {
        int64_t a = a0 + gemm_row(T::CL * wave + u);
        a = a < p.na ? a : p.na - 1;
        anc[u] = reinterpret_cast<const uint8_t*>(p.K + a * p.delta * p.GD + 8 * gemm_piece());
    }
    const int64_t jump = reinterpret_cast<const uint8_t*>(p.V) - reinterpret_cast<const uint8_t*>(p.K) - 2 * (int64_t)p.GD;
    const int steps = 2 * p.GD / 64;
    f32x4 acc[CF][TF];                        // [anchor tile][token tile] of this wave
    gemm_tile<TF, CF, false>(smem, tok, anc, jump, steps, acc);
    // the lane's anchors and their norms (absent anchors, numbers na and up: NaN keys, behind
    // every real anchor's, of which there are at least four)
    float nrm[CF][4];
#pragma unroll
    for (int j = 0; j < CF; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t a = a0 + 16 * (CF * wa + j) + 4 * grp + v;
            nrm[j][v] = a < p.na ? p.nrm[a] : NAN;
        }
    double* xt = reinterpret_cast<double*>(smem);              // [wt][TF token tiles][16][4]
    const uint32_t an = (uint32_t)(a0 + 16 * CF * wa + 4 * grp);
#pragma unroll
    for (int c = 0; c < TF; ++c) {
        Top4 t;
#pragma unroll
        for (int j = 0; j < CF; ++j) {
            Top4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t a = an + 16 * j + v;
                o[v] = anc_pack(nrm[j][v] - 2.f * acc[j][c][v], a);
            }
            top4_sort(o);
            if (j == 0) {
#pragma unroll
                for (int q = 0; q < AN_C; ++q) t[q] = o[q];
            } else {
                top4_merge(t, o);
            }
        }
        top4_lanes<16>(t);
        top4_lanes<32>(t);
        // lane group g of the token's four holds entry g
        const double mine = grp == 0 ? t[0] : grp == 1 ? t[1] : grp == 2 ? t[2] : t[3];
        if (wa == 1) {
            xt[((wt * TF + c) * 16 + col) * AN_C + grp] = mine;
        } else {
            acc[0][c] = __builtin_bit_cast(f32x4, (double2){t[0], t[1]});
            acc[1][c] = __builtin_bit_cast(f32x4, (double2){t[2], t[3]});
        }
    }
    __syncthreads();
    if (wa == 1) return;
#pragma unroll
    for (int c = 0; c < TF; ++c) {
        const double2 lo = __builtin_bit_cast(double2, acc[0][c]), hi = __builtin_bit_cast(double2, acc[1][c]);
        Top4 t = {lo.x, lo.y, hi.x, hi.y}, o;
        const int slot = ((wt * TF + c) * 16 + col) * AN_C;
#pragma unroll
        for (int q = 0; q < AN_C; ++q) o[q] = xt[slot + q];
        top4_merge(t, o);
        const int64_t i = i0 + 16 * (TF * wt + c) + col;
        const double mine = grp == 0 ? t[0] : grp == 1 ? t[1] : grp == 2 ? t[2] : t[3];
        if (i < p.Nc) p.part[((int64_t)at * p.Nc + i) * AN_C + grp] = mine;
    }
}

// ---- merge of the partial lists: one thread per coded token, all of a batch's loads in flight
__global__ __launch_bounds__(256) void anc_merge(const double* __restrict__ part, int64_t Nc, int n_atiles,
                                                uint16_t* __restrict__ nn) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= Nc) return;
    Top4 t;
#pragma unroll
    for (int q = 0; q < AN_C; ++q) t[q] = __builtin_bit_cast(double, AN_NONE);
    for (int at = 0; at < n_atiles; at += 4) {
        u32x4 w[4][2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double* src = part + ((int64_t)(at + k < n_atiles ? at + k : at) * Nc + i) * AN_C;
            w[k][0] = load16(src);
            w[k][1] = load16(src + 2);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (at + k >= n_atiles) break;
            const double2 lo = __builtin_bit_cast(double2, w[k][0]), hi = __builtin_bit_cast(double2, w[k][1]);
            const Top4 o = {lo.x, lo.y, hi.x, hi.y};
            top4_merge(t, o);
        }
    }
    uint2 out;
    out.x = pack2(anc_number(t[0]) & 0xFFFFu, anc_number(t[1]) & 0xFFFFu);
    out.y = pack2(anc_number(t[2]) & 0xFFFFu, anc_number(t[3]) & 0xFFFFu);
    anc_near_out(nn + i * AN_C, out);
}

// ---- compaction, residuals and the anchor store.  A workgroup per (64 rows, head), 16 lanes
// per 256-byte row piece and 8 elements per lane; rows: coded tokens i < Nc (residual), window
// rows (copied), anchors (copied).  Consecutive workgroups take consecutive heads, so with 8 (or
// 4) heads one XCD gathers the anchors of one head (512 KB at 2046 anchors) from its L2.  Bound
// by the K and V it reads and the residuals it writes: 118 us for the 32768-token Llama layer
// with 2-byte accesses and all heads on every XCD, 55 us now.  It also clears the list counts.
constexpr int AP_ROWS = 64;
__global__ __launch_bounds__(256) void anc_prep(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                                               const float* __restrict__ sbar, const uint16_t* __restrict__ nn,
                                               int64_t N, int64_t Nc, int64_t na, int w, int G, int delta,
                                               float* __restrict__ sbar_c, uint16_t* __restrict__ Kr,
                                               uint16_t* __restrict__ Vr, uint16_t* __restrict__ Ka,
                                               uint16_t* __restrict__ Va, uint32_t* __restrict__ cnt) {
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid < na) cnt[gid] = 0u;
    const int g = blockIdx.x % G;
    const int64_t r0 = (int64_t)(blockIdx.x / G) * AP_ROWS + (threadIdx.x >> 4);
    const int e = g * D + 8 * (threadIdx.x & 15);
    const int GD = G * D;
    const int64_t rows = Nc + w + na;
    uint2 near[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t r = r0 + 16 * k;
        near[k] = anc_near(nn + (r < Nc ? r : 0) * AN_C);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t r = r0 + 16 * k;
        if (r < Nc) {
            const int64_t t = anc_token(r, delta);
            const int64_t ta[AN_C] = {(int64_t)(near[k].x & 0xFFFFu) * delta, (int64_t)(near[k].x >> 16) * delta,
                                      (int64_t)(near[k].y & 0xFFFFu) * delta, (int64_t)(near[k].y >> 16) * delta};
            u32x4 x[2], m[2][AN_C];
            x[0] = load16(K + t * GD + e);
            x[1] = load16(V + t * GD + e);
#pragma unroll
            for (int q = 0; q < AN_C; ++q) {
                m[0][q] = load16(K + ta[q] * GD + e);
                m[1][q] = load16(V + ta[q] * GD + e);
            }
#pragma unroll
            for (int kv = 0; kv < 2; ++kv) {
                u32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float lo = 0.f, hi = 0.f;                    // fixed order: nearest first
#pragma unroll
                    for (int q = 0; q < AN_C; ++q) {
                        lo += bf_lo(m[kv][q][i]);
                        hi += bf_hi(m[kv][q][i]);
                    }
                    o[i] = cvt_bf16x2(bf_lo(x[kv][i]) - lo * (1.f / AN_C), bf_hi(x[kv][i]) - hi * (1.f / AN_C));
                }
                *reinterpret_cast<u32x4*>((kv ? Vr : Kr) + r * GD + e) = o;
            }
            if (e == 0) sbar_c[r] = sbar[t];
        } else if (r < rows) {
            const bool win = r < Nc + w;
            const int64_t a = r - Nc - w, t = win ? N + (r - Nc) : a * delta;
            const u32x4 xk = load16(K + t * GD + e), xv = load16(V + t * GD + e);
            *reinterpret_cast<u32x4*>((win ? Kr + r * GD : Ka + a * GD) + e) = xk;
            *reinterpret_cast<u32x4*>((win ? Vr + r * GD : Va + a * GD) + e) = xv;
        }
    }
}

// ---- after the allocation: anchors of every stored position, and the inverse lists.  Hub
// anchors are among the nearest of a large share of the tokens, so their counts and cursors are
// kept per workgroup of 1024 tokens in LDS and meet in memory once per workgroup and anchor
// (atomics of every token on them took 27 and 28 us for 30K tokens; 4.7 and 6.6 now).
// Past AL_LDS anchors the counts do not fit LDS and lists are short: one atomic per entry.
constexpr int AL_T = 1024;
constexpr int64_t AL_LDS = 12288;

template <bool LDS>
__global__ __launch_bounds__(AL_T) void anc_count(const uint32_t* __restrict__ sidx, const uint16_t* __restrict__ nn,
                                                 int64_t Nc, int64_t na, uint16_t* __restrict__ snn,
                                                 uint32_t* __restrict__ cnt) {
    extern __shared__ uint32_t hist[];
    const int tid = threadIdx.x;
    const int64_t p = (int64_t)blockIdx.x * AL_T + tid;
    const int64_t i = sidx[p < Nc ? p : Nc - 1];
    if constexpr (LDS) {
        for (int64_t a = tid; a < na; a += AL_T) hist[a] = 0u;
        __syncthreads();
    }
    if (p < Nc) {
        const uint2 q = anc_near(nn + i * AN_C);
        anc_near_out(snn + p * AN_C, q);
        uint32_t* dst = LDS ? hist : cnt;
        atomicAdd(&dst[q.x & 0xFFFFu], 1u);
        atomicAdd(&dst[q.x >> 16], 1u);
        atomicAdd(&dst[q.y & 0xFFFFu], 1u);
        atomicAdd(&dst[q.y >> 16], 1u);
    }
    if constexpr (LDS) {
        __syncthreads();
        for (int64_t a = tid; a < na; a += AL_T)
            if (hist[a]) atomicAdd(&cnt[a], hist[a]);
    }
}

template <bool LDS>
__global__ __launch_bounds__(AL_T) void anc_fill(const uint16_t* __restrict__ snn, int64_t Nc, int64_t na,
                                                uint32_t* __restrict__ cur, uint32_t* __restrict__ inv) {
    extern __shared__ uint32_t hist[];
    const int tid = threadIdx.x;
    const int64_t p = (int64_t)blockIdx.x * AL_T + tid;
    const bool in = p < Nc;
    const uint2 q = anc_near(snn + (in ? p : 0) * AN_C);
    const uint32_t a4[AN_C] = {q.x & 0xFFFFu, q.x >> 16, q.y & 0xFFFFu, q.y >> 16};
    if constexpr (LDS) {
        uint32_t slot[AN_C];
        for (int64_t a = tid; a < na; a += AL_T) hist[a] = 0u;
        __syncthreads();
        if (in)
#pragma unroll
            for (int k = 0; k < AN_C; ++k) slot[k] = atomicAdd(&hist[a4[k]], 1u);
        __syncthreads();
        // the workgroup's place in each list it adds to
        for (int64_t a = tid; a < na; a += AL_T)
            if (hist[a]) hist[a] = atomicAdd(&cur[a], hist[a]);
        __syncthreads();
        if (in)
#pragma unroll
            for (int k = 0; k < AN_C; ++k) inv[hist[a4[k]] + slot[k]] = (uint32_t)p;
    } else if (in) {
#pragma unroll
        for (int k = 0; k < AN_C; ++k) inv[atomicAdd(&cur[a4[k]], 1u)] = (uint32_t)p;
    }
}

// One workgroup between the two: the exclusive scan of the counts into the list starts (the
// counts become fill cursors, set to the starts), and the lists cut into pieces of 64 entries
// (hub anchors have long lists): the scan of the pieces, and each piece's anchor.  A thread takes
// consecutive anchors; anchors of more than 4 pieces are filled by their whole wave.
__global__ __launch_bounds__(AL_T) void anc_lists(uint32_t* __restrict__ cnt, int64_t na, uint32_t* __restrict__ off,
                                                 uint32_t* __restrict__ poff, uint16_t* __restrict__ panchor) {
    __shared__ uint2 wsum[AL_T / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t per = (na + AL_T - 1) / AL_T;
    const int64_t b0 = tid * per, b1 = b0 + per < na ? b0 + per : na;
    uint32_t s = 0, ps = 0;
    for (int64_t a = b0; a < b1; ++a) {
        const uint32_t c = cnt[a];
        s += c;
        ps += (c + 63) / 64;
    }
    uint32_t x = s, px = ps;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64), py = (uint32_t)__shfl_up((int)px, o, 64);
        if (lane >= o) { x += y; px += py; }
    }
    if (lane == 63) wsum[wave] = make_uint2(x, px);
    __syncthreads();
    uint32_t run = x - s, prun = px - ps, all = 0, pall = 0;
#pragma unroll
    for (int w = 0; w < AL_T / 64; ++w) {
        const uint2 v = wsum[w];
        run += w < wave ? v.x : 0u;
        prun += w < wave ? v.y : 0u;
        all += v.x;
        pall += v.y;
    }
    for (int64_t k = 0; k < per; ++k) {               // the same trip count in every lane
        const int64_t a = b0 + k;
        const uint32_t c = a < b1 ? cnt[a] : 0u, np = (c + 63) / 64;
        if (a < b1) {
            off[a] = run;
            cnt[a] = run;
            poff[a] = prun;
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (u < np) panchor[prun + u] = (uint16_t)a;
        for (unsigned long long hubs = __builtin_amdgcn_ballot_w64(np > 4); hubs; hubs &= hubs - 1) {
            const int l = __builtin_ctzll(hubs);
            const uint32_t p0 = (uint32_t)__builtin_amdgcn_readlane((int)prun, l);
            const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)np, l);
            const uint32_t ha = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, l);
            for (uint32_t u = 4 + lane; u < n; u += 64) panchor[p0 + u] = (uint16_t)ha;
        }
        run += c;
        prun += np;
    }
    if (tid == 0) {
        off[na] = all;
        poff[na] = pall;
    }
}

// ----------------------------------------------------------------------------------------
static inline int anc_atiles(const varrate_shape& sh) { return (int)((anchor_count(sh) + AN_TA - 1) / AN_TA); }

size_t anchor_ws_bytes(const varrate_shape& sh) {
    const int64_t Np = sh.n - sh.w, Nc = coded_count(sh), na = anchor_count(sh);
    const size_t rows = (size_t)(Nc + sh.w) * sh.G * D * 2;
    return align256(salience_ws_bytes(sh)) + align256(allocate_ws_bytes(sh)) + align256((size_t)Np * 4) +
           align256((size_t)Nc * 4) + align256((size_t)na * 4) + align256((size_t)anc_atiles(sh) * Nc * AN_C * 8) +
           align256((size_t)Nc * AN_C * 2) + 2 * align256(rows) + align256((size_t)na * 4);
}

AnchorWs anchor_ws(const varrate_shape& sh, uint8_t* ws) {
    const int64_t Np = sh.n - sh.w, Nc = coded_count(sh), na = anchor_count(sh);
    const size_t rows = (size_t)(Nc + sh.w) * sh.G * D * 2;
    AnchorWs w;
    uint8_t* p = ws;
    w.sal = p;                p += align256(salience_ws_bytes(sh));
    w.alloc = p;              p += align256(allocate_ws_bytes(sh));
    w.sbar = (float*)p;       p += align256((size_t)Np * 4);
    w.sbar_c = (float*)p;     p += align256((size_t)Nc * 4);
    w.nrm = (float*)p;        p += align256((size_t)na * 4);
    w.part = (double*)p;      p += align256((size_t)anc_atiles(sh) * Nc * AN_C * 8);
    w.nn = (uint16_t*)p;      p += align256((size_t)Nc * AN_C * 2);
    w.Kr = p;                 p += align256(rows);
    w.Vr = p;                 p += align256(rows);
    w.cnt = (uint32_t*)p;
    return w;
}

template <int TF, int CF>
static hipError_t launch_search(AnSearch& p, hipStream_t st) {
    typedef GemmTile<TF, CF, false> T;
    static_assert(T::LDS >= 4 * TF * 16 * AN_C * 8, "the halves' lists fit the stages");
    static_assert(T::ROWS >= AN_TA, "the workspace holds every tile's lists");
    p.n_atiles = (int)((p.na + T::ROWS - 1) / T::ROWS);
    p.n_ttiles = (int)((p.Nc + T::TOK - 1) / T::TOK);
    const int64_t per_xcd = ((int64_t)p.n_ttiles * p.n_atiles + 7) / 8;
    const hipError_t e = ensure_lds_limit((const void*)anc_search<TF, CF>, T::LDS);
    if (e != hipSuccess) return e;
    anc_search<TF, CF><<<(unsigned)(8 * per_xcd), 512, T::LDS, st>>>(p);
    return hipGetLastError();
}

hipError_t launch_anchor_search(const varrate_shape& sh, const void* K, const void* V, uint16_t* nn,
                                const AnchorWs& w, hipStream_t st) {
    const int64_t Nc = coded_count(sh), na = anchor_count(sh);
    const int GD = sh.G * D;
    anc_norms<<<(unsigned)((na + 3) / 4), 256, 0, st>>>((const uint16_t*)K, (const uint16_t*)V, na,
                                                        sh.anchor_stride, GD, w.nrm);
    AnSearch p;
    p.K = (const uint16_t*)K;
    p.V = (const uint16_t*)V;
    p.nrm = w.nrm;
    p.part = w.part;
    p.Nc = Nc;
    p.na = na;
    p.delta = sh.anchor_stride;
    p.GD = GD;
    // 256 x 256 tiles do the most per LDS byte, but one fills a CU where two of 64 tokens x 128
    // anchors share it: narrow ones are the faster as long as two rounds of 512 hold them all.
    // Whole compressions with either shape forced, narrow / wide us: 4 KV heads 126 / 129 at 864
    // narrow tiles, 143 / 144 at 1020, 155 / 151 at 1080, 134 / 129 at 1134; 8 KV heads 142 / 148,
    // 166 / 169, 178 / 169, 161 / 152.  Up to 256 anchors, one wide tile, nothing is read again from a
    // cache and three quarters of the CUs have to load: 8 KV heads, 157 anchors, 295 / 306 at 156 wide
    // tiles and 371 / 352 at 194; 98 anchors, one tile of either shape, 355 / 362 at 194
    const int64_t t64 = (Nc + 63) / 64, t256 = (Nc + 255) / 256;
    const bool wide = t64 * ((na + 127) / 128) > 1024 && (na > 256 || t256 >= 192);
    hipError_t e = wide ? launch_search<4, 8>(p, st) : launch_search<1, 4>(p, st);
    if (e != hipSuccess) return e;
    anc_merge<<<(unsigned)((Nc + 255) / 256), 256, 0, st>>>(w.part, Nc, p.n_atiles, nn);
    return hipGetLastError();
}

hipError_t launch_anchor_encode(const varrate_shape& sh, const void* K, const void* V, const float* sbar,
                                const uint16_t* nn, const float* PK, const float* PV, varrate_cache& c,
                                const AnchorWs& w, hipStream_t st) {
    const int64_t Np = sh.n - sh.w, Nc = coded_count(sh), na = anchor_count(sh);
    const varrate_shape shc = coded_shape(sh);
    const int64_t rows = Nc + sh.w + na;
    // one workgroup per 64 rows and head: more threads than anchors, whose counts they clear
    anc_prep<<<(unsigned)((rows + AP_ROWS - 1) / AP_ROWS * sh.G), 256, 0, st>>>(
        (const uint16_t*)K, (const uint16_t*)V, sbar, nn, Np, Nc, na, sh.w, sh.G, sh.anchor_stride, w.sbar_c,
        (uint16_t*)w.Kr, (uint16_t*)w.Vr, (uint16_t*)c.k_anchor, (uint16_t*)c.v_anchor, w.cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t* csz = nullptr;
    if ((e = launch_allocate(shc, w.sbar_c, c, w.alloc, st, nullptr, &csz)) != hipSuccess) return e;
    if ((e = launch_project(shc, w.Kr, w.Vr, PK, PV, c, st, csz)) != hipSuccess) return e;
    const unsigned wgs = (unsigned)((Nc + AL_T - 1) / AL_T);
    const size_t lds = na <= AL_LDS ? (size_t)na * 4 : 0;
    if (lds) anc_count<true><<<wgs, AL_T, lds, st>>>(c.sidx, nn, Nc, na, c.snn, w.cnt);
    else anc_count<false><<<wgs, AL_T, 0, st>>>(c.sidx, nn, Nc, na, c.snn, w.cnt);
    anc_lists<<<1, AL_T, 0, st>>>(w.cnt, na, c.inv_off, c.piece_off, c.piece_anchor);
    if (lds) anc_fill<true><<<wgs, AL_T, lds, st>>>(c.snn, Nc, na, w.cnt, c.inv_pos);
    else anc_fill<false><<<wgs, AL_T, 0, st>>>(c.snn, Nc, na, w.cnt, c.inv_pos);
    return hipGetLastError();
}

}  // namespace vr
