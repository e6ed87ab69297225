// Shared cross-head basis (Sec. 3.1 Eq. (1) "Joint per-token vector" and "Shared basis";
// Eq. (3) in joint units; Eq. (6)), gfx950.
//
// A token's keys and values of all G heads form z_t = [k_t; v_t] (Dz = 2 G d entries), coded
// against one basis W [R][Dz]: c_t = W z_t truncated to its rank, one coefficient row for
// every head and both K and V, stored in original token order (token t's row at offset[t]).
//
// Compress: the salience and allocation passes of the per-head codec (cap R, 16-bit ranks,
// per-token offsets, and per block of 128 coefficients the tokens that keep any of them), then
// C = Z W^T by bf16 MFMA with W split into bf16 hi + lo parts: jgemm_kernel over the token lists
// (bf16 layers, Z exact in bf16), jproj_kernel over consecutive tokens (fp32 layers, Z split too).
#include "vr_gemm.h"
#include "vr_internal.h"

namespace vr {

// ---- projection of fp32 layers -------------------------------------------------------------
constexpr int JP_T = 512;
constexpr int JP_TOK = 256;      // tokens per workgroup: 32 per wave (two 16-token blocks)
constexpr int JP_COL = 128;      // coefficients per workgroup: 8 blocks of 16

__global__ __launch_bounds__(JP_T, 2) void jproj_kernel(const float* __restrict__ K, const float* __restrict__ V,
                                                        const float* __restrict__ W,
                                                        const uint16_t* __restrict__ rank,
                                                        const uint32_t* __restrict__ offset, float* __restrict__ coef,
                                                        int64_t N, int G, int R) {
    __shared__ __attribute__((aligned(16))) u32x4 wl[2][2][8][64];   // [buffer][hi, lo][block][lane]
    __shared__ uint32_t s_max;
    const int half = G * D, Dz = 2 * G * D;
    const int nb = R / JP_COL;
    const int tb = blockIdx.x / nb, cb = blockIdx.x % nb;
    const int64_t t_base = (int64_t)tb * JP_TOK;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, col = lane & 15, grp = lane >> 4;
    // skip the workgroup when no token of its 256 keeps any of its 128 coefficients
    if (tid == 0) s_max = 0u;
    __syncthreads();
    if (tid < JP_TOK && t_base + tid < N) atomicMax(&s_max, (uint32_t)rank[t_base + tid]);
    __syncthreads();
    const int j_base = cb * JP_COL;
    if ((int)s_max <= j_base) return;
    // this wave's tokens: t_base + 32 wave + 16 mb + col (A rows); the stores' tokens below
    int64_t ta[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const int64_t t = t_base + 32 * wave + 16 * mb + col;
        ta[mb] = t < N ? t : N - 1;
    }
    // W staging: thread -> (block tid >> 6, lane): coefficient j_base + 16 (tid >> 6) + (lane & 15),
    // z coordinates k0 + 8 grp .. + 7
    const float* wrow = W + (int64_t)(j_base + 16 * (tid >> 6) + col) * Dz + 8 * grp;
    auto load_w = [&](int k0, u32x4& a, u32x4& b) {
        a = load16(wrow + k0);
        b = load16(wrow + k0 + 4);
    };
    auto put_w = [&](int buf, const u32x4& a, const u32x4& b) {
        float x8[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) { x8[e] = __uint_as_float(a[e]); x8[4 + e] = __uint_as_float(b[e]); }
        u32x4 h, l;
        split8(x8, h, l);
        wl[buf][0][tid >> 6][lane] = h;
        wl[buf][1][tid >> 6][lane] = l;
    };
    // A fragments (z of the wave's tokens): 8 elements as two 16-byte pieces
    auto zsrc = [&](int64_t t, int k) -> const float* {
        return k < half ? K + t * half + k : V + t * half + (k - half);
    };
    u32x4 za[2][2];
    auto load_z = [&](int k0, u32x4 (&z)[2][2]) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const float* p = zsrc(ta[mb], k0 + 8 * grp);
            z[mb][0] = load16(p);
            z[mb][1] = load16(p + 4);
        }
    };
    f32x4 acc[2][8];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[mb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nsteps = Dz / 32;
    u32x4 wa, wb;
    load_w(0, wa, wb);
    load_z(0, za);
    put_w(0, wa, wb);
    for (int s = 0; s < nsteps; ++s) {
        __syncthreads();    // buffer s & 1 is written; every wave is done with buffer (s + 1) & 1
        u32x4 zn[2][2];
        const bool more = s + 1 < nsteps;
        if (more) {
            load_w(32 * (s + 1), wa, wb);
            load_z(32 * (s + 1), zn);
        }
        const int buf = s & 1;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            u32x4 ah, al;
            float x8[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { x8[e] = __uint_as_float(za[mb][0][e]); x8[4 + e] = __uint_as_float(za[mb][1][e]); }
            split8(x8, ah, al);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const u32x4 wh = wl[buf][0][b][lane], wlo = wl[buf][1][b][lane];
                acc[mb][b] = mfma(ah, wh, acc[mb][b]);
                acc[mb][b] = mfma(ah, wlo, acc[mb][b]);
                acc[mb][b] = mfma(al, wh, acc[mb][b]);
            }
        }
        if (more) {
            put_w(buf ^ 1, wa, wb);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) { za[mb][0] = zn[mb][0]; za[mb][1] = zn[mb][1]; }
        }
    }
    // C lane -> tokens 4 grp + v of block mb, coefficient j_base + 16 b + col
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t t = t_base + 32 * wave + 16 * mb + 4 * grp + v;
            if (t >= N) continue;
            const int r = rank[t];
            const uint32_t o = offset[t];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int j = j_base + 16 * b + col;
                if (j < r) coef[o + j] = acc[mb][b][v];
            }
        }
    }
}

// ---- projection of bf16 layers -------------------------------------------------------------
// Ranks are spiky: at 20% most 256-token blocks hold some token of rank 1024 while the average
// rank is about 400, so blocks of consecutive tokens compute 2.5 times the kept coefficients.
// The allocation's last pass therefore leaves, per block of 128 coefficients, the list of tokens
// that keep any of them (in token order), and a workgroup takes 64 TF tokens of one list; only
// the coefficients up to the next multiple of 128 are computed for nothing.  W is split once
// into bf16 hi and lo parts in fragment order (jprep_kernel), z rows are gathered straight into
// the stages.  The products and their order per coefficient are those of jproj_kernel.  MFMA
// bound: 32768-token Llama layer, R = 1024, 467 us (one tile per 256 consecutive tokens and 128
// coefficients) before, 127 us now (920 TFLOP/s of 117 GFLOP; 1.8 rounds of tiles over the CUs).
struct JProj {
    const uint16_t* K;
    const uint16_t* V;
    const uint8_t* Wf;           // [R / 128][Dz / 64][2 (32 elements)][8 tiles][hi, lo][64] 16-byte fragments
    const uint32_t* list;        // [R / 128][N]
    const uint32_t* list_n;      // [R / 128]
    const uint16_t* rank;
    const uint32_t* offset;
    uint16_t* coef;
    int64_t N;
    int G, nb;
};

template <int TF>
__global__ __launch_bounds__(512, 2) void jgemm_kernel(JProj p) {
    typedef GemmTile<TF, 8, true> T;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    // tiles of all lists, block-major; XCD x (workgroup id mod 8) takes the x-th eighth, so it
    // keeps one or two blocks of W (1 MB each) in its L2
    uint32_t cnt[8], total = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) cnt[b] = b < p.nb ? p.list_n[b] : 0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) total += (cnt[b] + T::TOK - 1) / T::TOK;
    const uint32_t per = (total + 7) / 8, L = blockIdx.x;
    uint32_t id = (L & 7) * per + (L >> 3);
    if ((L >> 3) >= per || id >= total) return;
    int cb = 0;
    uint32_t n = cnt[0];
#pragma unroll
    for (int b = 0; b < 7; ++b) {
        const uint32_t tiles = (cnt[b] + T::TOK - 1) / T::TOK;
        if (cb == b && id >= tiles) { id -= tiles; cb = b + 1; n = cnt[b + 1]; }
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int col = lane & 15, grp = lane >> 4, wc = wave >> 2, wt = wave & 3;
    const uint32_t* list = p.list + (int64_t)cb * p.N;
    const uint32_t i0 = id * T::TOK;
    const int half = p.G * D, steps = 2 * half / 64;
    const uint8_t* tok[T::TL];
#pragma unroll
    for (int u = 0; u < T::TL; ++u) {
        const uint32_t i = i0 + gemm_row(T::TL * wave + u);
        const int64_t t = list[i < n ? i : n - 1];
        tok[u] = reinterpret_cast<const uint8_t*>(p.K + t * half + 8 * gemm_piece());
    }
    const uint8_t* wsrc[T::CL];
#pragma unroll
    for (int u = 0; u < T::CL; ++u)
        wsrc[u] = p.Wf + (int64_t)cb * steps * (128 * T::ROWS) + (T::CL * wave + u) * 1024 + lane * 16;
    const int64_t jump = reinterpret_cast<const uint8_t*>(p.V) - reinterpret_cast<const uint8_t*>(p.K) - 2 * (int64_t)half;
    f32x4 acc[4][TF];
    gemm_tile<TF, 8, true>(smem, tok, wsrc, jump, steps, acc);
    // lane -> token col of each fragment, coefficients 128 cb + 64 wc + 16 j + 4 grp + v
#pragma unroll
    for (int c = 0; c < TF; ++c) {
        const uint32_t i = i0 + 16 * (TF * wt + c) + col;
        if (i >= n) continue;
        const uint32_t t = list[i];
        const int r = p.rank[t];
        uint16_t* dst = p.coef + p.offset[t];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 128 * cb + 64 * wc + 16 * j + 4 * grp;
            if (k + 4 <= r) {
                const uint2 w = {pack2(f32_to_bf16(acc[j][c][0]), f32_to_bf16(acc[j][c][1])),
                                   pack2(f32_to_bf16(acc[j][c][2]), f32_to_bf16(acc[j][c][3]))};
                __builtin_memcpy(dst + k, &w, 8);            // 2-byte aligned
            } else {
#pragma unroll
                for (int v = 0; v < 3; ++v)
                    if (k + v < r) dst[k + v] = (uint16_t)f32_to_bf16(acc[j][c][v]);
            }
        }
    }
}

// One launch before the projection: W (fp32) into bf16 hi and lo fragments (bf16 layers), and the
// window rows, which stay exact: dst[g][e] = src[N + e][g] for K and V, 16 bytes per thread.
__global__ __launch_bounds__(256) void jprep_kernel(const float* __restrict__ W, u32x4* __restrict__ Wf, int w_wgs,
                                                    int Dz, const uint8_t* __restrict__ K, const uint8_t* __restrict__ V,
                                                    uint8_t* __restrict__ kx, uint8_t* __restrict__ vx, int64_t N, int G,
                                                    int w, int64_t cap, int row_bytes) {
    if ((int)blockIdx.x < w_wgs) {
        // (column tile, 32 elements)
        const int f = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, n32 = Dz / 32;
        const int ct = f / n32, k = f % n32;
        const float* src = W + (int64_t)(16 * ct + (lane & 15)) * Dz + 32 * k + 8 * (lane >> 4);
        const u32x4 a = load16(src), b = load16(src + 4);
        float x8[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) { x8[e] = __uint_as_float(a[e]); x8[4 + e] = __uint_as_float(b[e]); }
        u32x4 h, l;
        split8(x8, h, l);
        u32x4* dst = Wf + (((int64_t)(ct >> 3) * n32 + k) * 16 + (ct & 7) * 2) * 64 + lane;
        dst[0] = h;
        dst[64] = l;
        return;
    }
    const int upr = row_bytes / 16;
    const int64_t gid = (int64_t)(blockIdx.x - w_wgs) * 256 + threadIdx.x;
    const int64_t total = 2 * (int64_t)w * G * upr;
    if (gid >= total) return;
    const int kv = (int)(gid / ((int64_t)w * G * upr));
    const int64_t r = gid % ((int64_t)w * G * upr);
    const int e = (int)(r / (G * upr)), g = (int)((r / upr) % G), u = (int)(r % upr);
    const uint8_t* src = (kv ? V : K) + ((N + e) * G + g) * (int64_t)row_bytes + 16 * u;
    uint8_t* dst = (kv ? vx : kx) + ((int64_t)g * cap + e) * row_bytes + 16 * u;
    *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(src);
}

// Workspace of the projection: W's fragments, the token lists, the chunks' counts per block.
size_t joint_project_ws_bytes(const varrate_shape& sh, int R) {
    if (sh.dtype != VARRATE_BF16) return 0;
    const int64_t N = sh.n - sh.w;
    return align256((size_t)R * 2 * sh.G * D * 4) + align256((size_t)(R / 128) * N * 4) +
           align256((size_t)((N + CHUNK - 1) / CHUNK) * 16) + 256;
}
JointLists joint_lists(const varrate_shape& sh, int R, uint8_t* ws) {
    JointLists l = {nullptr, nullptr, nullptr, 0};
    if (sh.dtype != VARRATE_BF16) return l;
    const int64_t N = sh.n - sh.w;
    uint8_t* p = ws + align256((size_t)R * 2 * sh.G * D * 4);
    l.list = (uint32_t*)p;    p += align256((size_t)(R / 128) * N * 4);
    l.ccnt = (uint4*)p;       p += align256((size_t)((N + CHUNK - 1) / CHUNK) * 16);
    l.list_n = (uint32_t*)p;
    l.nb = R / 128;
    return l;
}

// 256-token tiles reuse W best, but one fills a CU where two of the 64-token tiles share it: up to
// 128 wide tiles the 512 or fewer narrow ones all run at once and are the faster, and so they are
// (from 8 KV heads on: 32 steps a tile) where wide tiles leave a second round that is less than a
// quarter full.  The lists' lengths are known on the device only; estimated here as B / 128 rows,
// 5/8 of a row for every token below the cap R, and half a tile per list.  Whole compressions with
// either shape forced (R = 256 and 1024, 10 to 40%, 1K to 32K tokens), narrow / wide us: 4 KV heads
// 104 / 118 at 84 wide tiles, 118 / 128 at 112, 129 / 126 at 140, 146 / 134 at 240, 172 / 170 at 292, 166 / 161 at 360; 8 KV heads
// 103 / 121 at 114, 107 / 121 at 124, 129 / 123 at 149, 143 / 130 at 238, 167 / 175 at 266,
// 181 / 184 at 295, 189 / 187 at 355, 233 / 201 at 473.  By tokens instead (wide past 12288)
// R = 256 lost up to 18 us at 16384 tokens.
static bool joint_wide(int64_t N, int64_t B, int R, int G) {
    const int64_t tiles = (B / 128 + (N - B / R) * 5 / 8) / 256 + R / 256;
    return tiles > 128 && (tiles <= 256 || tiles > 320 || G < 8);
}

template <int TF>
static hipError_t launch_jgemm(const JProj& p, hipStream_t st) {
    typedef GemmTile<TF, 8, true> T;
    const hipError_t e = ensure_lds_limit((const void*)jgemm_kernel<TF>, T::LDS);
    if (e != hipSuccess) return e;
    // room for every list at its longest; workgroups past the lists' tiles end at once
    const int64_t tiles = (p.N + T::TOK - 1) / T::TOK * p.nb;
    jgemm_kernel<TF><<<(unsigned)((tiles + 7) / 8 * 8), 512, T::LDS, st>>>(p);
    return hipGetLastError();
}

hipError_t launch_joint_project(const varrate_shape& sh, int R, const void* K, const void* V, const float* W,
                                varrate_jcache& c, uint8_t* ws, hipStream_t st) {
    const int64_t N = sh.n - sh.w;
    const bool bf16 = sh.dtype == VARRATE_BF16;
    const int row_bytes = D * (bf16 ? 2 : 4), Dz = 2 * sh.G * D;
    const int w_wgs = bf16 ? (R / 16) * (Dz / 32) / 4 : 0;
    const int64_t units = 2 * (int64_t)sh.w * sh.G * (row_bytes / 16);
    jprep_kernel<<<(unsigned)(w_wgs + (units + 255) / 256), 256, 0, st>>>(W, (u32x4*)ws, w_wgs, Dz, (const uint8_t*)K,
                                                                          (const uint8_t*)V, (uint8_t*)c.k_exact,
                                                                          (uint8_t*)c.v_exact, N, sh.G, sh.w, c.cap,
                                                                          row_bytes);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!bf16) {
        const unsigned blocks = (unsigned)(((N + JP_TOK - 1) / JP_TOK) * (R / JP_COL));
        jproj_kernel<<<blocks, JP_T, 0, st>>>((const float*)K, (const float*)V, W, c.rank, c.offset, (float*)c.coef, N,
                                              sh.G, R);
        return hipGetLastError();
    }
    const JointLists l = joint_lists(sh, R, ws);
    JProj p;
    p.K = (const uint16_t*)K;
    p.V = (const uint16_t*)V;
    p.Wf = ws;
    p.list = l.list;
    p.list_n = l.list_n;
    p.rank = c.rank;
    p.offset = c.offset;
    p.coef = (uint16_t*)c.coef;
    p.N = N;
    p.G = sh.G;
    p.nb = l.nb;
    return joint_wide(N, c.B, R, sh.G) ? launch_jgemm<4>(p, st) : launch_jgemm<1>(p, st);
}

}  // namespace vr
