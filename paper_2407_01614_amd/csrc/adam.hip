// Partition step: Adam(W) over one rank's flat fp32 shard, emitting the bf16
// primary shard (optimizer.step() of Algorithm 1 on the rank's partition).
//
// Pure streaming work: 16 B read + 14 B written per element and about 45
// VALU operations (correctly rounded sqrt and division included), so HBM
// bandwidth is the bound.  Each thread owns U float4 groups per tile; a wave's
// load instruction covers 1 KiB of one array, all 4*U loads of a tile are
// issued before any arithmetic, and every access is non-temporal (nothing is
// reused).  The grid is one-shot (one tile per workgroup): on this GPU a
// persistent grid of a few thousand workgroups streams about 20% slower.
// Residency is capped at ZPP_ADAM_RESIDENCY one-wave workgroups per CU: at
// the Llama-2-13B partition the step takes 923-931 us with 10 resident
// (928-944 with 9 or 11), 1003-1016 us uncapped.
#include "zpp_adam.h"
#include "zpp_device.h"
#include "zpp_launch.h"

#ifndef ZPP_ADAM_UNROLL
#define ZPP_ADAM_UNROLL 1
#endif
#ifndef ZPP_ADAM_THREADS
#define ZPP_ADAM_THREADS 64
#endif
#ifndef ZPP_ADAM_RESIDENCY
#define ZPP_ADAM_RESIDENCY 10
#endif

namespace zpp {
namespace {

struct AdamArgs {
    float *p, *m, *v;
    const float *g;
    uint16_t *out;
    AdamConsts c;
};

constexpr int kAdamThreads = ZPP_ADAM_THREADS;

template <bool ADAMW, int U, bool WHOLE>
__device__ __forceinline__ void adam_tile(const AdamArgs &a, size_t base, uint32_t rest) {
    f32x4 P[U], M[U], V[U], G[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = (u * kAdamThreads + threadIdx.x) * 4;
        P[u] = load4<WHOLE>(a.p + base, i, rest);
        M[u] = load4<WHOLE>(a.m + base, i, rest);
        V[u] = load4<WHOLE>(a.v + base, i, rest);
        G[u] = load4<WHOLE>(a.g + base, i, rest);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = (u * kAdamThreads + threadIdx.x) * 4;
        adam_update4<ADAMW>(P[u], M[u], V[u], G[u], a.c);
        store4<WHOLE>(a.p + base, i, rest, P[u]);
        store4<WHOLE>(a.m + base, i, rest, M[u]);
        store4<WHOLE>(a.v + base, i, rest, V[u]);
        store4_bf16<WHOLE>(a.out + base, i, rest,
                           u32x2{pack_bf16x2(P[u].x, P[u].y), pack_bf16x2(P[u].z, P[u].w)});
    }
}

template <bool ADAMW, int U>
__global__ __launch_bounds__(kAdamThreads) void adam_vec_kernel(AdamArgs a, TileSpan tiles) {
    constexpr uint32_t kTile = kAdamThreads * 4 * U;
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, tiles, 0);
    const size_t base = (tiles.first + t) * kTile;
    if (__builtin_expect(t < tiles.whole, 1))
        adam_tile<ADAMW, U, true>(a, base, kTile);
    else
        adam_tile<ADAMW, U, false>(a, base, tiles.tail);
}

}  // namespace

hipError_t launch_adam(float *p, float *m, float *v, const float *g, uint16_t *out, size_t n,
                       const AdamConsts &c, bool on_lines, hipStream_t stream) {
    const AdamArgs a{p, m, v, g, out, c};
    constexpr uint32_t kTile = kAdamThreads * 4 * ZPP_ADAM_UNROLL;
    const size_t lds = launch_lds(ZPP_ADAM_RESIDENCY, n / kTile);
    for_tiles(n, kTile, 1, kAdamThreads, on_lines, [&](const TileSpan &tiles, unsigned grid) {
        if (c.adamw)
            hipLaunchKernelGGL((adam_vec_kernel<true, ZPP_ADAM_UNROLL>), dim3(grid),
                               dim3(kAdamThreads), lds, stream, a, tiles);
        else
            hipLaunchKernelGGL((adam_vec_kernel<false, ZPP_ADAM_UNROLL>), dim3(grid),
                               dim3(kAdamThreads), lds, stream, a, tiles);
    });
    return hipGetLastError();
}

}  // namespace zpp
