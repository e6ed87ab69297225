// Group-wise b-bit quantisation of a compressed layer's coefficients (Sec. 3.3
// "Composability": the coefficients are quantised on their own, the allocation unchanged).
//
// Groups: one stored position's coefficients of one head and stream (K or V) in one
// 32-coordinate segment.  Symmetric absmax per group: with Qmax = 2^(b-1) - 1,
//     sc = binary16(fp32(amax / Qmax)),   k = clamp(rint(fp32(x / sc)), -Qmax, Qmax),
// correctly rounded fp32 divisions, ties to even; a group with sc = 0 codes 0.  The input x
// is the stored bf16 coefficient; entries past a position's rank are stored zeros, so they
// change neither amax nor their code (0).
//
// Output layout, per head stream, tile by tile in the same storage order as the coefficient
// layout (chunk c at qchunk_off[c] bytes): a tile of size m (its first position's rank)
// takes mq = m rounded up to a multiple of 8 coordinates and KS = ceil(m / 32) groups per
// position:
//   K stream: 16 rows of mq codes (code (i, j) at bit b (i mq + j)), then KS x 16 scales;
//   V stream: mq rows of 16 codes (code (j, i) at bit b (16 j + i)), then KS x 16 scales;
// codes are two's complement b-bit fields from bit 0 of the tile upward, scales binary16
// at [s][position].  Tile bytes: 2 mq b + 32 KS (a multiple of 16).
//
// Two launches: one workgroup sums the tile sizes of every chunk and scans them into
// qchunk_off; then a workgroup per (chunk, head, stream) writes that chunk's tiles.
#include "vr_internal.h"

namespace vr {

constexpr int QZ_SCAN_THREADS = 1024;

__host__ __device__ constexpr uint32_t qz_tile_bytes(uint32_t m, int b) {
    return m == 0 ? 0u : 2u * ((m + 7u) & ~7u) * (uint32_t)b + 32u * ((m + 31u) / 32u);
}

// Chunk offsets: a thread takes one tile (one rank byte) per pass, all of a pass's loads
// independent, and the 16 lanes of a chunk add up by a row reduction; the chunk sums of up to
// QZ_SCAN_CHUNKS chunks then go through one scan.  Latency is all it costs: with one thread
// walking 16 dependent rank loads per chunk it took 7.4 us at 30K tokens, now 4.5.
constexpr int QZ_SCAN_CHUNKS = QZ_SCAN_THREADS;       // chunks per scan block

// sum over the 16 lanes of a row, in every lane
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);   // row_ror:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, true);
    return v;
}
// inclusive sum over the lanes of a row up to this one
__device__ __forceinline__ uint32_t row_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1, zeros shifted in
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    return v;
}

__global__ __launch_bounds__(QZ_SCAN_THREADS) void qz_scan_kernel(const uint8_t* __restrict__ srank,
                                                                  int64_t N, int n_chunks, int bits,
                                                                  uint32_t* __restrict__ qchunk_off) {
    __shared__ uint32_t part[QZ_SCAN_CHUNKS];
    __shared__ uint32_t wsum[QZ_SCAN_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t base = 0;                                   // bytes of the scan blocks before
    for (int cb = 0; cb < n_chunks; cb += QZ_SCAN_CHUNKS) {
        const int nc = min(QZ_SCAN_CHUNKS, n_chunks - cb);
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int tile = QZ_SCAN_THREADS * k + tid;  // of this block; 16 tiles per chunk
            const int64_t i = 16 * ((int64_t)16 * cb + tile);
            const uint32_t b = row_sum(i < N ? qz_tile_bytes(srank[i], bits) : 0u);
            if ((lane & 15) == 0) part[tile >> 4] = b;   // chunks past the last one: 0
            if (QZ_SCAN_THREADS * (k + 1) >= 16 * nc) break;
        }
        __syncthreads();
        const uint32_t own = tid < nc ? part[tid] : 0u;
        uint32_t v = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)v, off, 64);
            if (lane >= off) v += o;
        }
        if (lane == 63) wsum[wave] = v;
        __syncthreads();
        uint32_t before = base, all = base;
#pragma unroll
        for (int w = 0; w < QZ_SCAN_THREADS / 64; ++w) {
            before += w < wave ? wsum[w] : 0u;
            all += wsum[w];
        }
        if (tid < nc) qchunk_off[cb + tid] = before + v - own;
        base = all;
        __syncthreads();                                 // part and wsum are reused
    }
    if (tid == 0) qchunk_off[n_chunks] = base;
}

struct QzParams {
    const uint16_t* coef[2];     // bf16 streams (K, V), [G][coef_stride]
    uint8_t* code[2];            // code streams (K, V), [G][q_stride] bytes
    const uint8_t* srank;
    const uint32_t* chunk_off;   // bf16 layout chunk bases (elements)
    const uint32_t* qchunk_off;  // quantised chunk bases (bytes)
    int64_t N, coef_stride, q_stride;
    int G;
};

// One workgroup per (chunk, head, stream), its wave w taking tiles w, w + 4, w + 8, w + 12.
// A wave quantises one 32-coordinate segment of a tile (16 positions x 32 coordinates, 1 KB of
// bf16) per step, straight from registers: 8 coefficients per lane, of one group in the K
// stream (position lane / 4, coordinates 8 (lane % 4) ..) and of one coordinate in the V
// stream (coordinate lane / 2, positions 8 (lane % 2) ..), which is how either stream stores
// them.  The first segments of all four tiles are requested before the first is used and a
// tile's next segment before its current one, so the step is bound by its VALU work: about 9
// instructions per coefficient (staging the tile and its codes in LDS, with a row / column
// split and a full division per element, took 75 us for the 29987-token layer where this
// takes 18).
//
// Arithmetic.  Absolute bf16 values order as their 15-bit patterns do, so a group's absmax is
// a packed integer maximum.  Both divisions are a product with a reciprocal and one residual
// correction.  amax / Qmax: the reciprocal is the constant's nearest fp32 value, so the
// corrected quotient is correctly rounded.  x / scale, for |x| <= amax with an 8-bit
// significand and a scale with at most 11 bits: a quotient that is not exactly half-way between
// two integers is at least 2^-12 away from it, far more than the error, and one that is
// exactly half-way comes out exact, so the rounding to an integer (the addition of
// 1.5 * 2^23, ties to even) agrees with that of the correctly rounded quotient.  Groups whose
// scale is not finite (absmax above the binary16 range, infinities, NaN) take the plain
// divisions.
constexpr int QZ_WAVES = 4;

__device__ __forceinline__ uint32_t qz_umax2(uint32_t a, uint32_t b) {     // packed 16-bit maxima
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 x = __builtin_bit_cast(u16x2, a), y = __builtin_bit_cast(u16x2, b);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(x, y));
}
template <int CTRL> __device__ __forceinline__ uint32_t qz_dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// binary16 scale of a group from its absmax (finite)
template <int QB> __device__ __forceinline__ _Float16 qz_scale(float amax) {
    constexpr float Q = (float)((1 << (QB - 1)) - 1), RQ = 1.0f / Q;
    const float q = amax * RQ;
    return (_Float16)fmaf(fmaf(-q, Q, amax), RQ, q);
}
// code of x at scale sc with rc = 1 / sc (both 0 for a zero group), in the low bits
template <int QB> __device__ __forceinline__ uint32_t qz_code(float x, float sc, float rc) {
    constexpr float Q = (float)((1 << (QB - 1)) - 1);
    const float q0 = x * rc;
    const float q = fmaf(fmaf(-q0, sc, x), rc, q0);
    return __float_as_uint(__builtin_amdgcn_fmed3f(q, -Q, Q) + 12582912.f);
}
// the same by the plain divisions (any sc)
template <int QB> __device__ __forceinline__ uint32_t qz_code_any(float x, float sc) {
    constexpr float Q = (float)((1 << (QB - 1)) - 1);
    if (sc == 0.f) return 0u;
    return (uint32_t)(int)fminf(fmaxf(__builtin_rintf(__fdiv_rn(x, sc)), -Q), Q);
}
// 8 codes (low bits of c[k]) -> 8 QB bits at dst (any byte address)
template <int QB> __device__ __forceinline__ void qz_store(uint8_t* dst, const uint32_t (&c)[8]) {
    if constexpr (QB == 8) {
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k >> 2] = __builtin_amdgcn_alignbit(c[k], w[k >> 2], 8);
        *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
    } else {
        uint32_t w = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) w = __builtin_amdgcn_alignbit(c[k], w, QB);
        if constexpr (QB == 4) {
            *reinterpret_cast<uint32_t*>(dst) = w;
        } else {
            w >>= 8;
            dst[0] = (uint8_t)w;
            dst[1] = (uint8_t)(w >> 8);
            dst[2] = (uint8_t)(w >> 16);
        }
    }
}

template <int QB>
__global__ __launch_bounds__(64 * QZ_WAVES) void qz_kernel(QzParams p) {
    constexpr int NT = 16 / QZ_WAVES;             // tiles per wave
    constexpr uint32_t INF16 = 0x7F80u;           // bf16 infinity's pattern
    __shared__ __attribute__((aligned(16))) float scl_s[QZ_WAVES][2][16];   // V: scales, reciprocals
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int item = blockIdx.x;                  // (chunk, head, stream)
    const int kv = item & 1;
    const int g = (item >> 1) % p.G;
    const int c = (item >> 1) / p.G;
    const int64_t t0 = (int64_t)c * CHUNK;
    const int T = (int)(p.N - t0 < CHUNK ? p.N - t0 : CHUNK);
    const int ntile = (T + 15) >> 4;
    // lane h < 16: tile h's size and its offsets within the chunk (absent tiles: size 0)
    const uint32_t mlane = (lane & 15) < ntile ? (uint32_t)p.srank[t0 + 16 * (lane & 15)] : 0u;
    const uint32_t eo = row_scan(16u * mlane) - 16u * mlane;
    const uint32_t tb = qz_tile_bytes(mlane, QB);
    const uint32_t bo = row_scan(tb) - tb;
    const uint16_t* base_src = p.coef[kv] + (int64_t)g * p.coef_stride + p.chunk_off[c];
    uint8_t* base_dst = p.code[kv] + (int64_t)g * p.q_stride + p.qchunk_off[c];
    // this lane's 8 coefficients of segment s of a tile of size m (zeros past the tile)
    auto fetch = [&](const uint16_t* src, int m, int s) -> u32x4 {
        if (kv == 0) {
            const int j = 32 * s + 8 * (lane & 3);
            if (j >= m) return u32x4{0u, 0u, 0u, 0u};
            return load16_a2(src + (lane >> 2) * m + j);     // may run past the row: masked below
        }
        if (32 * s + (lane >> 1) >= m) return u32x4{0u, 0u, 0u, 0u};
        return load16(src + 512 * s + 8 * lane);
    };
    int mt[NT];
    u32x4 first[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int h = wave + QZ_WAVES * k;
        mt[k] = __builtin_amdgcn_readlane((int)mlane, h);
        first[k] = fetch(base_src + __builtin_amdgcn_readlane((int)eo, h), mt[k], 0);
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int h = wave + QZ_WAVES * k, m = mt[k];
        const int mq = (m + 7) & ~7, ks = (m + 31) / 32;
        const uint16_t* src = base_src + __builtin_amdgcn_readlane((int)eo, h);
        uint8_t* dst = base_dst + __builtin_amdgcn_readlane((int)bo, h);
        uint16_t* sdst = reinterpret_cast<uint16_t*>(dst + 2 * mq * QB);
        u32x4 next = first[k];
        for (int s = 0; s < ks; ++s) {
            u32x4 x = next;
            if (s + 1 < ks) next = fetch(src, m, s + 1);
            uint32_t code[8];
            if (kv == 0) {
                const int i = lane >> 2, j = 32 * s + 8 * (lane & 3);
                const int nv = m - j;
                x = keep_first(x, nv < 0 ? 0 : (nv > 8 ? 8 : nv));
                const u32x4 ab = x & 0x7FFF7FFFu;
                uint32_t mx = qz_umax2(qz_umax2(ab[0], ab[1]), qz_umax2(ab[2], ab[3]));
                mx = qz_umax2(mx, mx >> 16) & 0xFFFFu;
                mx = max(mx, qz_dpp<0xB1>(mx));              // quad_perm [1,0,3,2]
                mx = max(mx, qz_dpp<0x4E>(mx));              // quad_perm [2,3,0,1]
                _Float16 hs = qz_scale<QB>(__uint_as_float(mx << 16));
                const bool odd = mx >= INF16 || (float)hs == INFINITY;
                if (__builtin_amdgcn_ballot_w64(odd) == 0) {
                    const float sc = (float)hs, rc = sc != 0.f ? __builtin_amdgcn_rcpf(sc) : 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) code[e] = qz_code<QB>((e & 1) ? bf_hi(x[e >> 1]) : bf_lo(x[e >> 1]), sc, rc);
                } else {
                    float amax = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((e & 1) ? bf_hi(x[e >> 1]) : bf_lo(x[e >> 1])));
                    amax = fmaxf(amax, __shfl_xor(amax, 1, 64));
                    amax = fmaxf(amax, __shfl_xor(amax, 2, 64));
                    hs = (_Float16)__fdiv_rn(amax, (float)((1 << (QB - 1)) - 1));
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        code[e] = qz_code_any<QB>((e & 1) ? bf_hi(x[e >> 1]) : bf_lo(x[e >> 1]), (float)hs);
                }
                if (j < mq) qz_store<QB>(dst + (i * mq + j) / 8 * QB, code);
                if ((lane & 3) == 0) sdst[16 * s + i] = __builtin_bit_cast(uint16_t, hs);
            } else {
                // absmax of the lane's 8 positions over the 32 coordinates (the lanes of its
                // parity): the two swaps halve what a lane holds, so it ends with the dword
                // (two positions) 2 (lane / 32) + (lane / 16) % 2 of its parity's four
                const u32x4 ab = x & 0x7FFF7FFFu;
                const auto e0 = __builtin_amdgcn_permlane32_swap(ab[0], ab[2], false, false);
                const auto e1 = __builtin_amdgcn_permlane32_swap(ab[1], ab[3], false, false);
                const auto e2 = __builtin_amdgcn_permlane16_swap(qz_umax2(e0[0], e0[1]), qz_umax2(e1[0], e1[1]), false, false);
                uint32_t mx = qz_umax2(e2[0], e2[1]);
                mx = qz_umax2(mx, qz_dpp<0x128>(mx));        // row_ror: 8, 4, 2
                mx = qz_umax2(mx, qz_dpp<0x124>(mx));
                mx = qz_umax2(mx, qz_dpp<0x122>(mx));
                const int p0 = 8 * (lane & 1) + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1);
                _Float16 h0 = qz_scale<QB>(__uint_as_float(mx << 16)), h1 = qz_scale<QB>(__uint_as_float(mx & 0xFFFF0000u));
                const bool odd = (mx & 0xFFFFu) >= INF16 || (mx >> 16) >= INF16 || (float)h0 == INFINITY || (float)h1 == INFINITY;
                const bool plain = __builtin_amdgcn_ballot_w64(odd) == 0;
                float* scl = scl_s[wave][0];
                float* rcp = scl_s[wave][1];
                if (plain) {
                    if ((lane & 14) == 0) {
                        const float s0 = (float)h0, s1 = (float)h1;
                        *reinterpret_cast<float2*>(scl + p0) = make_float2(s0, s1);
                        *reinterpret_cast<float2*>(rcp + p0) = make_float2(s0 != 0.f ? __builtin_amdgcn_rcpf(s0) : 0.f,
                                                                           s1 != 0.f ? __builtin_amdgcn_rcpf(s1) : 0.f);
                        *reinterpret_cast<uint32_t*>(sdst + 16 * s + p0) =
                            pack2(__builtin_bit_cast(uint16_t, h0), __builtin_bit_cast(uint16_t, h1));
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    f32x4 sc[2], rc[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        sc[q] = *reinterpret_cast<const f32x4*>(scl + 8 * (lane & 1) + 4 * q);
                        rc[q] = *reinterpret_cast<const f32x4*>(rcp + 8 * (lane & 1) + 4 * q);
                    }
                    __builtin_amdgcn_wave_barrier();         // the next step writes them again
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        code[e] = qz_code<QB>((e & 1) ? bf_hi(x[e >> 1]) : bf_lo(x[e >> 1]), sc[e >> 2][e & 3], rc[e >> 2][e & 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float v = (e & 1) ? bf_hi(x[e >> 1]) : bf_lo(x[e >> 1]);
                        float amax = fmaxf(0.f, fabsf(v));
#pragma unroll
                        for (int off = 2; off < 64; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
                        const _Float16 hs = (_Float16)__fdiv_rn(amax, (float)((1 << (QB - 1)) - 1));
                        code[e] = qz_code_any<QB>(v, (float)hs);
                        if (lane < 2) sdst[16 * s + 8 * lane + e] = __builtin_bit_cast(uint16_t, hs);
                    }
                }
                const int j = 32 * s + (lane >> 1);
                if (j < mq) qz_store<QB>(dst + (16 * j + 8 * (lane & 1)) / 8 * QB, code);
            }
        }
    }
}

// ----------------------------------------------------------------------------------------
size_t qcache_stride(const varrate_shape& sh, int bits) {
    const int64_t N = coded_count(sh);
    const int64_t n_chunks = (N + CHUNK - 1) / CHUNK;
    const int64_t B = coded_budget(sh);
    // a chunk's tile maxima sum to at most its ranks / 16 + 128, each tile pads up to 7
    // coordinates and holds at most 4 groups per position
    const int64_t bound = (int64_t)bits * B / 8 + n_chunks * (480LL * bits + 2048) + 64;
    return (size_t)((bound + 15) / 16 * 16);
}

hipError_t launch_quantize(const varrate_shape& sh, const varrate_cache& c, varrate_qcache& q, hipStream_t st) {
    const int64_t N = coded_count(sh);
    const int n_chunks = (int)((N + CHUNK - 1) / CHUNK);
    qz_scan_kernel<<<1, QZ_SCAN_THREADS, 0, st>>>(c.srank, N, n_chunks, q.bits, q.qchunk_off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    QzParams p;
    p.coef[0] = (const uint16_t*)c.coef_k;
    p.coef[1] = (const uint16_t*)c.coef_v;
    p.code[0] = (uint8_t*)q.code_k;
    p.code[1] = (uint8_t*)q.code_v;
    p.srank = c.srank;
    p.chunk_off = c.chunk_off;
    p.qchunk_off = q.qchunk_off;
    p.N = N;
    p.coef_stride = c.coef_stride;
    p.q_stride = q.q_stride;
    p.G = sh.G;
    const int grid = n_chunks * sh.G * 2;                       // (chunk, head, stream)
    switch (q.bits) {
        case 3: qz_kernel<3><<<grid, 64 * QZ_WAVES, 0, st>>>(p); break;
        case 4: qz_kernel<4><<<grid, 64 * QZ_WAVES, 0, st>>>(p); break;
        case 8: qz_kernel<8><<<grid, 64 * QZ_WAVES, 0, st>>>(p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace vr
