// Tile product shared by the shared-basis projection and the nearest-anchor search (gfx950; its
// direct-to-LDS load also serves the shared-basis decode):
// C[column][token] = sum over Dz of col[c][k] z_t[k], bf16 MFMA with fp32 sums, in steps of 64
// elements of z.
//
// Workgroup: 8 waves, 64 TF tokens against 32 CF rows of the column operand; wave (wc, wt) =
// (wave / 4, wave % 4) multiplies its CF 16-row column fragments (A operand) with its TF
// 16-token fragments (B operand).  Both operands come by direct-to-LDS loads of 1 KB, all of a
// stage's loads spread evenly over the waves, NS stages rotating behind one barrier a step:
//   rows (tokens; columns when !FRAG): 8 rows x 128 bytes per load, so every request is a whole
//       128-byte line; row r's 16-byte piece c lies at place c ^ (r % 8), which makes the
//       fragment reads (16 rows, one piece each) free of bank conflicts;
//   FRAG: columns as bf16 hi and lo parts already in fragment order, contiguous per step.
//
// What bounds it: 64-byte requests (16 rows x 32 elements per load) cap the loads at about half of
// what the matrix cores can use: 620 TFLOP/s for 256 x 128 tiles of 30720 x 2048 x 2048, 740 with
// the products left out.  Whole lines give 1460 with the products left out, 1440 with the loads
// left out and 1230 together (a library's plain product of that size, second operand transposed
// as here: 1325; of 8192^3: 1650).
#pragma once
#include "vr_device.h"

namespace vr {

template <int TF, int CF, bool FRAG>
struct GemmTile {
    static constexpr int TOK = 64 * TF;                       // tokens per workgroup
    static constexpr int ROWS = 32 * CF;                      // column-operand rows (FRAG: both parts)
    static constexpr int TILES = FRAG ? CF / 2 : CF;          // 16-column tiles per wave
    static constexpr int STAGE = (TOK + ROWS) * 128;
    static constexpr int TL = TF, CL = CF / 2;                // loads per wave and stage
    static constexpr int NS = 3 * STAGE <= 80 * 1024 ? 3 : 2;
    static constexpr size_t LDS = (size_t)NS * STAGE;
    static_assert(LDS <= 160 * 1024 && CF % 2 == 0, "stages fit one CU, whole loads per wave");
};

// One direct-to-LDS load: 16 bytes per lane from `src` to LDS byte address dst + 16 lane.
__device__ __forceinline__ void gemm_load(const void* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst) : "memory", "m0");
}

// The row (of the workgroup's tile) and 16-byte piece that this lane brings with load f.
__device__ __forceinline__ int gemm_row(int f) { return 8 * f + ((threadIdx.x & 63) >> 3); }
__device__ __forceinline__ int gemm_piece() { return (threadIdx.x & 7) ^ ((threadIdx.x & 63) >> 3); }

// tok[u]: this lane's source of token load TL wave + u at step 0, advancing 128 bytes a step and
// by `jump` bytes more from step steps / 2 on (the value half of z).  col[u]: the same for
// column load CL wave + u; FRAG: advancing 128 ROWS bytes a step instead, no jump.
template <int TF, int CF, bool FRAG>
__device__ __forceinline__ void gemm_tile(uint8_t* smem, const uint8_t* (&tok)[TF], const uint8_t* (&col)[CF / 2],
                                          int64_t jump, int steps,
                                          f32x4 (&acc)[GemmTile<TF, CF, FRAG>::TILES][TF]) {
    typedef GemmTile<TF, CF, FRAG> T;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int wc = wave >> 2, wt = wave & 3, l16 = lane & 15, grp = lane >> 4;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem);
    int is = 0;                               // next step to issue
    uint32_t ibuf = lds0;                     // its stage
    auto issue = [&]() {
#pragma unroll
        for (int u = 0; u < T::TL; ++u) {
            gemm_load(tok[u], ibuf + 1024u * (uint32_t)(T::TL * wave + u));
            tok[u] += 128;
        }
#pragma unroll
        for (int u = 0; u < T::CL; ++u) {
            gemm_load(col[u], ibuf + 1024u * (uint32_t)(8 * TF + T::CL * wave + u));
            col[u] += FRAG ? 128 * T::ROWS : 128;
        }
        ++is;
        if (2 * is == steps) {
#pragma unroll
            for (int u = 0; u < T::TL; ++u) tok[u] += jump;
            if constexpr (!FRAG)
#pragma unroll
                for (int u = 0; u < T::CL; ++u) col[u] += jump;
        }
        ibuf += T::STAGE;
        if (ibuf == lds0 + (uint32_t)T::NS * T::STAGE) ibuf = lds0;
    };
#pragma unroll
    for (int j = 0; j < T::TILES; ++j)
#pragma unroll
        for (int c = 0; c < TF; ++c) acc[j][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < T::NS - 1 && s < steps; ++s) issue();
    const uint8_t* rbuf = smem;
    for (int s = 0; s < steps; ++s) {
        // stage s has landed when at most the loads of the stage after it are in flight
        constexpr int PER = T::TL + T::CL;
        static_assert(T::NS == 2 || PER == 3, "immediate wait count below");
        if (T::NS == 3 && s + 1 < steps) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                      // every wave's part of stage s; stage s - 1 is free
        if (is < steps) issue();
        const uint8_t* cbuf = rbuf + T::TOK * 128;
#pragma unroll
        for (int h = 0; h < 2; ++h) {         // 32 elements each
            const int place = ((4 * h + grp) ^ (l16 & 7)) * 16;
            u32x4 ft[TF], fc[CF];
#pragma unroll
            for (int c = 0; c < TF; ++c)
                ft[c] = *reinterpret_cast<const u32x4*>(rbuf + (16 * (TF * wt + c) + l16) * 128 + place);
            if constexpr (FRAG) {
#pragma unroll
                for (int j = 0; j < CF; ++j)  // (tile, part) pairs
                    fc[j] = *reinterpret_cast<const u32x4*>(cbuf + ((h * 2 * CF + CF * wc + j) * 64 + lane) * 16);
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int j = 0; j < T::TILES; ++j)
#pragma unroll
                        for (int c = 0; c < TF; ++c) acc[j][c] = mfma(fc[2 * j + q], ft[c], acc[j][c]);
            } else {
#pragma unroll
                for (int j = 0; j < CF; ++j)
                    fc[j] = *reinterpret_cast<const u32x4*>(cbuf + (16 * (CF * wc + j) + l16) * 128 + place);
#pragma unroll
                for (int j = 0; j < CF; ++j)
#pragma unroll
                    for (int c = 0; c < TF; ++c) acc[j][c] = mfma(fc[j], ft[c], acc[j][c]);
            }
        }
        rbuf += T::STAGE;
        if (rbuf == smem + (size_t)T::NS * T::STAGE) rbuf = smem;
    }
    __syncthreads();                          // every wave is done with the stages
}

}  // namespace vr
