// Secondary refresh: bit copy of the local rank's bf16 weights into the hpZ
// secondary partition (Algorithm 1, forward loop; Eq. 1).  2 B read + 2 B
// written per element.  Each thread moves U 16-byte vectors per tile, all
// loads issued before the stores, non-temporal both ways.  Shape, swept at
// the Llama-2-13B partition (813 MB moved): one-wave workgroups with one
// vector per lane, residency left to the hardware, 120.7-123.1 us; four-wave
// workgroups with four vectors per lane 124.3-131.1 us, capped or not.
#include "zpp_device.h"
#include "zpp_launch.h"

#ifndef ZPP_REFRESH_UNROLL
#define ZPP_REFRESH_UNROLL 1
#endif
#ifndef ZPP_REFRESH_THREADS
#define ZPP_REFRESH_THREADS 64
#endif
#ifndef ZPP_REFRESH_RESIDENCY
#define ZPP_REFRESH_RESIDENCY 0
#endif

namespace zpp {
namespace {

constexpr int kRefreshThreads = ZPP_REFRESH_THREADS;

// One tile of 512 U elements; the lanes of a partial tile's last vector go
// element by element, all loads before the stores.
template <int U>
__global__ __launch_bounds__(kRefreshThreads) void refresh_vec_kernel(
    uint16_t *__restrict__ dst, const uint16_t *__restrict__ src, TileSpan tiles) {
    constexpr uint32_t kTile = kRefreshThreads * 8 * U;  // 8 bf16 per 16-byte vector
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, tiles, 0);
    dst += (tiles.first + t) * kTile;
    src += (tiles.first + t) * kTile;
    if (__builtin_expect(t < tiles.whole, 1)) {
        u32x4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[u] = ld_nt_at<u32x4, 2>(src + (u * kRefreshThreads + threadIdx.x) * 8);
#pragma unroll
        for (int u = 0; u < U; ++u)
            st_nt_at<u32x4, 2>(dst + (u * kRefreshThreads + threadIdx.x) * 8, x[u]);
    } else {
        uint16_t x[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[u][e] = src[clamped((u * kRefreshThreads + threadIdx.x) * 8 + e, tiles.tail)];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t i = (u * kRefreshThreads + threadIdx.x) * 8 + e;
                if (i < tiles.tail)
                    dst[i] = x[u][e];
            }
    }
}

}  // namespace

hipError_t launch_refresh(uint16_t *dst, const uint16_t *src, size_t count, bool on_lines,
                          hipStream_t stream) {
    for_tiles(count, kRefreshThreads * 8 * ZPP_REFRESH_UNROLL, 1, kRefreshThreads, on_lines,
              [&](const TileSpan &tiles, unsigned grid) {
                  hipLaunchKernelGGL((refresh_vec_kernel<ZPP_REFRESH_UNROLL>), dim3(grid),
                                     dim3(kRefreshThreads), residency_lds(ZPP_REFRESH_RESIDENCY),
                                     stream, dst, src, tiles);
              });
    return hipGetLastError();
}

}  // namespace zpp
