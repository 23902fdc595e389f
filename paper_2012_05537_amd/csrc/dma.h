// Staging of population rows in LDS by DMA copies (no register holds the data).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sllbm {

// DMA copies of 16 and 4 bytes per lane from g into LDS at l + size * lane (l is
// wave-uniform).  AUX is the copy's cache-policy operand (2: non-temporal, 0:
// the default policy).  Untyped, in device functions of their own: the 16-byte
// form exists on gfx950 only, and the host pass drops the launch stub of a
// kernel whose body names it.
template <int AUX>
__device__ __forceinline__ void dma16(const void *g, void *l)
{
    __builtin_amdgcn_global_load_lds(g, l, 16, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ void dma4(const void *g, void *l)
{
    __builtin_amdgcn_global_load_lds(g, l, 4, 0, AUX);
}

// Rows r = 0 .. ROWS - 1 (even) of in (stride N), columns nb .. nb + NB - 1, NB =
// 512 / sizeof(S), to tile, by the NW waves of a block; w is this wave, lane
// its lane.  Columns past N are left as they are.  WIDE: 16 bytes per lane, two
// rows (1 KB) per instruction, for N a multiple of 16 / sizeof(S) and in
// 16-byte aligned (a lane's values are then all below N or all beyond it);
// otherwise 4 bytes per lane, half a row per instruction.  Ends with this
// wave's copies landed; the caller's barrier covers the others'.
template <typename S, int ROWS, int NB, int NW, bool WIDE, bool NTH>
__device__ __forceinline__ void stage_rows(int64_t N, int64_t nb, const S *in, S (&tile)[ROWS][NB], int w, int lane)
{
    static_assert(NB * sizeof(S) == 512 && ROWS % 2 == 0, "row of 512 bytes");
    constexpr int AUX = NTH ? 2 : 0;
    if constexpr (WIDE) {
        const int64_t col = nb + static_cast<int>(16 / sizeof(S)) * (lane & 31);
        if (col < N) {
            const S *src = in + static_cast<int64_t>(lane >> 5) * N + col;
            for (int m = w; m < ROWS / 2; m += NW)
                dma16<AUX>(src + static_cast<int64_t>(2 * m) * N, &tile[2 * m][0]);
        }
    } else {
        constexpr int W = sizeof(S) / 4;                   // words per value
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int64_t word = nb * W + half * 64 + lane;
            if (word < N * W) {
                const uint32_t *src = reinterpret_cast<const uint32_t *>(in) + word;
                for (int r = w; r < ROWS; r += NW)
                    dma4<AUX>(src + static_cast<int64_t>(r) * N * W, &tile[r][half * (NB / 2)]);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
}

}  // namespace sllbm
