// qwZ quantization of a bf16 weight shard: symmetric absmax int8 per block of
// B elements with one fp32 scale per block (weights are quantized before the
// AllGather, Background section).  2 B read, 1 B + 4/B B written per element.
//
// Vector kernel: one lane holds 8 consecutive bf16 (one 16-byte load), so a
// block of B elements spans L = min(B/8, 64) lanes of one wave and a lane
// holds V = max(1, B/512) vectors.  The absmax is an integer max over the bf16
// magnitude bits (|x| bits are monotone in |x|, and bits >= 0x7F80 mean Inf or
// NaN), reduced across the L lanes with cross-lane xor shuffles; no LDS
// traffic and no float compares are needed.  Every lane then derives the
// block's scale and inverse itself (two correctly rounded divisions per 8
// elements) and writes its 8 codes as one 8-byte store.  Blocks that are
// not powers of two (any multiple of 64 up to 4096) take the same approach
// with the block's width a run-time value: a block owns an aligned group of
// 16 to 64 lanes, each holding up to 16 of its vectors.
//
// The same kernels can also store the bf16 they read to a second array:
// the secondary refresh and its quantization in one pass (2 B read, 2 B +
// 1 B + 4/B B written per element, against 4 + 3 + 4/B B for the two
// calls).
#include "zpp_chunk.h"
#include "zpp_device.h"
#include "zpp_launch.h"
#include "zpp_quant.h"

#ifndef ZPP_QUANT_UNROLL
#define ZPP_QUANT_UNROLL 2
#endif
#ifndef ZPP_QUANT_THREADS
#define ZPP_QUANT_THREADS 256
#endif
// Shape of the kernel for blocks that are not powers of two (zpp_chunk.h):
// at least two vector slots per lane, and the widest lane group whose slots
// the block fills to this percentage.  Swept at the Llama-2-13B partition
// over blocks of 192 to 2112 (median of 20 launches each): the plain
// quantizer streams best with a fill of 75% (93-102 us against 97-120 for
// 55-85% or three slots), the pass with the copy with 55% (167-175 us
// against 168-185); one slot per lane was slower for both (137 against
// 97 us at 448).
#ifndef ZPP_QUANT_GROUP_MIN_FILL
#define ZPP_QUANT_GROUP_MIN_FILL 75
#endif
#ifndef ZPP_QUANT_COPY_GROUP_MIN_FILL
#define ZPP_QUANT_COPY_GROUP_MIN_FILL 55
#endif
#ifndef ZPP_QUANT_MAX_GRID
#define ZPP_QUANT_MAX_GRID (1u << 20)
#endif
// Block-rows in flight per wave of the refresh-and-quantize pass: one, where
// the quantizer alone streams best with two (Llama-2-13B partition: 157.6
// against 164.8 us; the plain quantizer 112 against 94 us with one).
#ifndef ZPP_QUANT_COPY_UNROLL
#define ZPP_QUANT_COPY_UNROLL 1
#endif

namespace zpp {
namespace {

constexpr int kQuantThreads = ZPP_QUANT_THREADS;

// The workgroup's place in the array.  The pass with the copy takes runs of
// workgroups per XCD where its outputs do not start on lines, for the blocks
// and lengths of quant_copy_runs (zpp_chunk.h).  The quantizer alone gains
// nothing from them (10.0 us at 13.1 M without, 10.2 with).  RUNS is a template
// argument: chosen at run time it cost the pass on lines 0.7%.
template <bool RUNS>
__device__ __forceinline__ uint32_t group_of() {
    return RUNS ? (uint32_t)xcd_grouped(blockIdx.x, gridDim.x, kOffLineXcdRun) : blockIdx.x;
}

template <int B, int U>
__global__ __launch_bounds__(kQuantThreads) void quant_vec_kernel(
    const uint16_t *__restrict__ src, size_t n, int8_t *__restrict__ codes,
    float *__restrict__ scales) {
    constexpr int L = (B / 8 < kWave) ? B / 8 : kWave;  // lanes per quant block
    constexpr int V = (B / 8 > kWave) ? B / (8 * kWave) : 1;
    constexpr int kGroupsPerWave = kWave / L;
    constexpr int kGroupsPerRow = kGroupsPerWave * (kQuantThreads / kWave);
    constexpr int kGroupsPerBlock = kGroupsPerRow * U;
    const size_t nblocks = (n + B - 1) / B;
    const int lane = threadIdx.x & (kWave - 1);
    const int gl = lane / L;
    const int li = lane % L;
    const int wave = threadIdx.x / kWave;

    for (size_t g0 = (size_t)blockIdx.x * kGroupsPerBlock; g0 < nblocks;
         g0 += (size_t)gridDim.x * kGroupsPerBlock) {
        // all U rows of loads first, then the reductions and stores
        u32x4 x[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t k = g0 + (size_t)u * kGroupsPerRow + (size_t)wave * kGroupsPerWave + gl;
            const bool valid = k < nblocks;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const size_t i = k * B + ((size_t)v * L + li) * 8;
                if (valid && i + 8 <= n) {
                    x[u][v] = ld_nt_at<u32x4, 2>(src + i);
                } else {
                    uint32_t h[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        h[e] = (valid && i + e < n) ? (uint32_t)src[i + e] : 0u;
                    x[u][v] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16),
                                    h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t k = g0 + (size_t)u * kGroupsPerRow + (size_t)wave * kGroupsPerWave + gl;
            const bool valid = k < nblocks;
            u16x2 m2 = {0, 0};
#pragma unroll
            for (int v = 0; v < V; ++v)
                m2 = __builtin_elementwise_max(m2, __builtin_elementwise_max(
                         __builtin_elementwise_max(absbits2(x[u][v].x), absbits2(x[u][v].y)),
                         __builtin_elementwise_max(absbits2(x[u][v].z), absbits2(x[u][v].w))));
            uint32_t mx = max((uint32_t)m2.x, (uint32_t)m2.y);
#pragma unroll
            for (int off = L / 2; off >= 1; off >>= 1)
                mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));

            const BlockQuant q = block_params(mx);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const size_t i = k * B + ((size_t)v * L + li) * 8;
                u32x2 c;
                c.x = quant_word(x[u][v].x, x[u][v].y, q);
                c.y = quant_word(x[u][v].z, x[u][v].w, q);
                if (valid && i + 8 <= n) {
                    st_nt_at<u32x2, 1>(codes + i, c);
                } else if (valid) {
                    for (int e = 0; e < 8 && i + e < n; ++e)
                        codes[i + e] =
                            (int8_t)((e < 4 ? c.x >> (8 * e) : c.y >> (8 * (e - 4))) & 0xFFu);
                }
            }
            if (valid && li == 0)
                scales[k] = q.scale;
        }
    }
}

// The quantization with the copy: the workgroup's U rows of blocks, `rest`
// elements of them inside the arrays (WHOLE: all of them).
template <int B, int U, bool WHOLE>
__device__ __forceinline__ void quant_copy_rows(const uint16_t *__restrict__ src,
                                                int8_t *__restrict__ codes,
                                                float *__restrict__ scales,
                                                uint16_t *__restrict__ copy, uint32_t rest) {
    constexpr int L = (B / 8 < kWave) ? B / 8 : kWave;  // lanes per quant block
    constexpr int V = (B / 8 > kWave) ? B / (8 * kWave) : 1;
    constexpr int kGroupsPerWave = kWave / L;
    constexpr int kGroupsPerRow = kGroupsPerWave * (kQuantThreads / kWave);
    const uint32_t li = threadIdx.x % L;
    const uint32_t k0 = threadIdx.x / L;
    // all U rows of loads first, then the reductions and stores
    u32x4 x[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t i = (u * kGroupsPerRow + k0) * B + (v * L + li) * 8;
            if (WHOLE || i + 8 <= rest) {
                x[u][v] = ld_nt_at<u32x4, 2>(src + i);
            } else {
                uint32_t h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    h[e] = i + e < rest ? (uint32_t)src[i + e] : 0u;
                x[u][v] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                h[6] | (h[7] << 16)};
            }
        }
    const auto row = [&](int u) {
        const uint32_t k = u * kGroupsPerRow + k0;
        u16x2 m2 = {0, 0};
#pragma unroll
        for (int v = 0; v < V; ++v)
            m2 = __builtin_elementwise_max(m2, __builtin_elementwise_max(
                     __builtin_elementwise_max(absbits2(x[u][v].x), absbits2(x[u][v].y)),
                     __builtin_elementwise_max(absbits2(x[u][v].z), absbits2(x[u][v].w))));
        uint32_t mx = max((uint32_t)m2.x, (uint32_t)m2.y);
#pragma unroll
        for (int off = L / 2; off >= 1; off >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));

        const BlockQuant q = block_params(mx);
        const auto store = [&](int v) {
            const uint32_t i = k * B + (v * L + li) * 8;
            u32x2 c;
            c.x = quant_word(x[u][v].x, x[u][v].y, q);
            c.y = quant_word(x[u][v].z, x[u][v].w, q);
            if (WHOLE || i + 8 <= rest) {
                st_nt_at<u32x2, 1>(codes + i, c);
                st_nt_at<u32x4, 2>(copy + i, x[u][v]);
            } else {
                for (int e = 0; e < 8 && i + e < rest; ++e) {
                    codes[i + e] =
                        (int8_t)((e < 4 ? c.x >> (8 * e) : c.y >> (8 * (e - 4))) & 0xFFu);
                    copy[i + e] = src[i + e];
                }
            }
        };
        // no loop over a single vector (nor, below, over a single row): its
        // store would be hoisted out of it as a plain, temporal one (203 M
        // elements 164 us, 158 non-temporal)
        if constexpr (V == 1) {
            store(0);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v)
                store(v);
        }
        if (li == 0 && (WHOLE || k * B < rest))
            scales[k] = q.scale;
    };
    if constexpr (U == 1) {
        row(0);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
            row(u);
    }
}

// The loaded bf16 are also stored to `copy`, bit for bit (the secondary
// refresh taken into the quantization's pass).  Straight code for whole
// workgroups: 25.9 M elements 22.5 -> 22.1 us, 203 M 161.6 -> 158.4, blocks of
// 4096 177 -> 171.  (The quantizer alone written so is 5-15% faster up to 4 M
// elements and 4-7% slower from 13 M on, so it keeps its own form.)
template <int B, int U, bool RUNS>
__global__ __launch_bounds__(kQuantThreads) void quant_copy_kernel(
    const uint16_t *__restrict__ src, int8_t *__restrict__ codes, float *__restrict__ scales,
    uint16_t *__restrict__ copy, TileSpan tiles) {
    constexpr uint32_t C = (B < 512 ? 512 : B) * (kQuantThreads / kWave) * U;
    const uint32_t t = group_of<RUNS>();
    const size_t base = (tiles.first + t) * C;
    src += base;
    codes += base;
    scales += base / B;
    copy += base;
    if (__builtin_expect(t < tiles.whole, 1))
        quant_copy_rows<B, U, true>(src, codes, scales, copy, C);
    else
        quant_copy_rows<B, U, false>(src, codes, scales, copy, tiles.tail);
}

// Vector path for a block B = 64 b that is not a power of two, lane-group
// layout (zpp_chunk.h): each block owns an aligned group of G lanes, lane r
// of the group holding the block's vectors v G + r for v < S (vectors past
// the block's end stay empty), so a wave load covers 64 / G runs of G
// consecutive vectors.  The block absmax is a reduction over the group's G
// lanes with cross-lane xor shuffles and every lane derives the block's
// parameters itself, as in the power-of-two kernel: no LDS, no atomics and
// no barrier.  Workgroups whose blocks all lie inside the array load each
// vector with one predicated load; only the last one checks every element.
template <int G, int S, bool COPY, bool RUNS>
__global__ __launch_bounds__(kQuantThreads) void quant_grp_kernel(
    const uint16_t *__restrict__ src, size_t n, uint32_t B, int8_t *__restrict__ codes,
    float *__restrict__ scales, uint16_t *__restrict__ copy) {
    constexpr int kGroupsPerWave = kWave / G;
    constexpr int kGroupsPerBlock = kGroupsPerWave * (kQuantThreads / kWave);
    const uint32_t vpb = B / 8;
    const size_t nblocks = (n + B - 1) / B;
    const int lane = threadIdx.x & (kWave - 1);
    const int li = lane % G;
    const size_t kw = (size_t)(threadIdx.x / kWave) * kGroupsPerWave + lane / G;
    for (size_t g0 = (size_t)group_of<RUNS>() * kGroupsPerBlock; g0 < nblocks;
         g0 += (size_t)gridDim.x * kGroupsPerBlock) {
        const size_t k = g0 + kw;
        const bool valid = k < nblocks;
        const bool whole = (g0 + kGroupsPerBlock) * B <= n;  // uniform
        u32x4 x[S];
        if (whole) {
#pragma unroll
            for (int v = 0; v < S; ++v) {
                x[v] = u32x4{0u, 0u, 0u, 0u};
                const uint32_t j = (uint32_t)(v * G + li);
                if (j < vpb)
                    x[v] = ld_nt_at<u32x4, 2>(src + k * B + (size_t)j * 8);
            }
        } else {
#pragma unroll
            for (int v = 0; v < S; ++v) {
                x[v] = u32x4{0u, 0u, 0u, 0u};
                const uint32_t j = (uint32_t)(v * G + li);
                const size_t i = k * B + (size_t)j * 8;
                if (valid && j < vpb) {
                    if (i + 8 <= n) {
                        x[v] = ld_nt_at<u32x4, 2>(src + i);
                    } else if (i < n) {
                        uint32_t h[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            h[e] = (i + e < n) ? (uint32_t)src[i + e] : 0u;
                        x[v] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16),
                                     h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
                    }
                }
            }
        }
        u16x2 m2 = {0, 0};
#pragma unroll
        for (int v = 0; v < S; ++v)
            m2 = __builtin_elementwise_max(m2, __builtin_elementwise_max(
                     __builtin_elementwise_max(absbits2(x[v].x), absbits2(x[v].y)),
                     __builtin_elementwise_max(absbits2(x[v].z), absbits2(x[v].w))));
        uint32_t mx = max((uint32_t)m2.x, (uint32_t)m2.y);
#pragma unroll
        for (int off = G / 2; off >= 1; off >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        const BlockQuant q = block_params(mx);
#pragma unroll
        for (int v = 0; v < S; ++v) {
            const uint32_t j = (uint32_t)(v * G + li);
            const size_t i = k * B + (size_t)j * 8;
            if (!valid || j >= vpb || i >= n)
                continue;
            u32x2 c;
            c.x = quant_word(x[v].x, x[v].y, q);
            c.y = quant_word(x[v].z, x[v].w, q);
            if (i + 8 <= n) {
                st_nt_at<u32x2, 1>(codes + i, c);
                if (COPY)
                    st_nt_at<u32x4, 2>(copy + i, x[v]);
            } else {
                for (int e = 0; e < 8 && i + e < n; ++e) {
                    codes[i + e] =
                        (int8_t)((e < 4 ? c.x >> (8 * e) : c.y >> (8 * (e - 4))) & 0xFFu);
                    if (COPY)
                        copy[i + e] = src[i + e];
                }
            }
        }
        if (valid && li == 0)
            scales[k] = q.scale;
    }
}

template <int B, bool COPY>
void launch_vec(const uint16_t *src, size_t n, int8_t *codes, float *scales, uint16_t *copy,
                bool on_lines, hipStream_t stream) {
    constexpr int U = COPY ? ZPP_QUANT_COPY_UNROLL : ZPP_QUANT_UNROLL;
    constexpr uint32_t C = (B < 512 ? 512 : B) * (kQuantThreads / kWave) * U;
    if constexpr (COPY) {
        constexpr bool kRuns = B <= 512;  // quant_copy_runs
        for_tiles(n, C, 1, kQuantThreads, on_lines, [&](const TileSpan &tiles, unsigned grid) {
            if (kRuns && !on_lines)
                hipLaunchKernelGGL((quant_copy_kernel<B, U, kRuns>), dim3(grid),
                                   dim3(kQuantThreads), 0, stream, src, codes, scales, copy,
                                   tiles);
            else
                hipLaunchKernelGGL((quant_copy_kernel<B, U, false>), dim3(grid),
                                   dim3(kQuantThreads), 0, stream, src, codes, scales, copy,
                                   tiles);
        });
    } else {
        const size_t need = (n + C - 1) / C;
        const unsigned grid = (unsigned)(need < ZPP_QUANT_MAX_GRID ? need : ZPP_QUANT_MAX_GRID);
        hipLaunchKernelGGL((quant_vec_kernel<B, U>), dim3(grid), dim3(kQuantThreads), 0, stream,
                           src, n, codes, scales);
    }
}

template <int G, int S, bool COPY>
void launch_grp(const uint16_t *src, size_t n, uint32_t block, int8_t *codes, float *scales,
                uint16_t *copy, bool on_lines, hipStream_t stream) {
    constexpr size_t kGroupsPerBlock = (kWave / G) * (kQuantThreads / kWave);
    const size_t nblocks = (n + block - 1) / block;
    const size_t need = (nblocks + kGroupsPerBlock - 1) / kGroupsPerBlock;
    const unsigned grid = (unsigned)(need < ZPP_QUANT_MAX_GRID ? need : ZPP_QUANT_MAX_GRID);
    constexpr bool kRuns = COPY && S == 2;  // the blocks of quant_copy_runs
    if (kRuns && !on_lines && quant_copy_runs(block, n))
        hipLaunchKernelGGL((quant_grp_kernel<G, S, COPY, kRuns>), dim3(grid), dim3(kQuantThreads),
                           0, stream, src, n, block, codes, scales, copy);
    else
        hipLaunchKernelGGL((quant_grp_kernel<G, S, COPY, false>), dim3(grid), dim3(kQuantThreads),
                           0, stream, src, n, block, codes, scales, copy);
}

template <int S, bool COPY>
void launch_grp_g(uint32_t G, const uint16_t *src, size_t n, uint32_t block, int8_t *codes,
                  float *scales, uint16_t *copy, bool on_lines, hipStream_t stream) {
    switch (G) {
    case 16: launch_grp<16, S, COPY>(src, n, block, codes, scales, copy, on_lines, stream); break;
    case 32: launch_grp<32, S, COPY>(src, n, block, codes, scales, copy, on_lines, stream); break;
    default: launch_grp<64, S, COPY>(src, n, block, codes, scales, copy, on_lines, stream); break;
    }
}

template <bool COPY>
void launch_vector(const uint16_t *src, size_t n, uint32_t block, int8_t *codes, float *scales,
                   uint16_t *copy, bool on_lines, hipStream_t stream) {
    switch (block) {
    case 64: launch_vec<64, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 128: launch_vec<128, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 256: launch_vec<256, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 512: launch_vec<512, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 1024: launch_vec<1024, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 2048: launch_vec<2048, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    case 4096: launch_vec<4096, COPY>(src, n, codes, scales, copy, on_lines, stream); break;
    default: {
        const GroupShape sh =
            COPY ? group_shape(block / 8, 16, ZPP_QUANT_COPY_GROUP_MIN_FILL, 2)
                 : group_shape(block / 8, 16, ZPP_QUANT_GROUP_MIN_FILL, 2);
        if (sh.S <= 2)
            launch_grp_g<2, COPY>(sh.G, src, n, block, codes, scales, copy, on_lines, stream);
        else if (sh.S <= 4)
            launch_grp_g<4, COPY>(sh.G, src, n, block, codes, scales, copy, on_lines, stream);
        else if (sh.S <= 8)
            launch_grp_g<8, COPY>(sh.G, src, n, block, codes, scales, copy, on_lines, stream);
        else
            launch_grp_g<16, COPY>(sh.G, src, n, block, codes, scales, copy, on_lines, stream);
    }
    }
}

}  // namespace

hipError_t launch_quantize_copy(const uint16_t *src, size_t n, uint32_t block, int8_t *codes,
                                float *scales, uint16_t *copy, bool on_lines,
                                hipStream_t stream) {
    launch_vector<true>(src, n, block, codes, scales, copy, on_lines, stream);
    return hipGetLastError();
}

hipError_t launch_quantize(const uint16_t *src, size_t n, uint32_t block, int8_t *codes,
                           float *scales, hipStream_t stream) {
    launch_vector<false>(src, n, block, codes, scales, nullptr, true, stream);
    return hipGetLastError();
}

}  // namespace zpp
