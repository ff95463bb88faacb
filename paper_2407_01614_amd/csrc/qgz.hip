// qgZ, the gradient side of the partition step: blockwise int4 quantization
// of fp32 gradients before the exchange that replaces the ReduceScatter
// (Background section; Algorithm 1, backward loop), and, on the receiving
// rank, the dequantize-and-reduce of the P quantized copies of its partition
// into the fp32 gradient the optimizer step consumes.
//
// Quantize: 4 B read, 0.5 B + 4/B B written per element.  The absmax is an
// integer max of the |x| bit patterns (bits >= 0x7F800000 mean Inf or NaN),
// reduced over the lanes of a block with xor shuffles.  Codes come from the
// same round-to-nearest-even trick as the int8 quantizer (the low bits of
// x*inv + 1.5*2^23), packed four to a 16-bit store.
//
// Dequant-reduce: P * (0.5 B + 4/B B) read, 4 B written per element.  The
// sources' pointers travel by value in the kernel arguments; a lane
// accumulates its elements over the sources in order, one fma each.
//
// The dequant-reduce is one kernel over the gradient sources of the receive
// kernels (zpp_i4grad.h): the P copies as separate arrays or in one
// interleaved receive buffer, with the same bits.
//
// Blocks may be any multiple of 64 up to 4096; for those that are not powers
// of two the quantizer gives each block an aligned group of 16 to 64 lanes
// of a wave, each lane holding several of its groups of 4 values.
//
// The power-of-two kernels keep every wave's loads and stores contiguous: on
// this GPU, non-temporal stores that leave gaps inside a wave's footprint
// (16 bytes per lane at a 32- or 64-byte stride) run two to three times
// slower.  The lane-group quantizer's code stores are runs of 2 G bytes per
// block (32 to 128), which the sweep of its shapes measured: groups of 8
// lanes (16-byte runs) were the slow ones and are not used.
#include "zpp_chunk.h"
#include "zpp_device.h"
#include "zpp_i4grad.h"
#include "zpp_launch.h"
#include "zpp_quant.h"

#ifndef ZPP_QGZ_THREADS
#define ZPP_QGZ_THREADS 256
#endif
// Shape of the quantizer for blocks that are not powers of two
// (zpp_chunk.h): at least three slots per lane, and the widest lane group
// whose slots the block fills to this percentage.  Swept at the Llama-2-13B
// partition over blocks of 192 to 4032 (median of 20 launches each): 149-157
// us with this rule, against up to 173 us with two slots and 220 with
// groups of 8 lanes (16-byte runs of codes per store instruction), and
// 191-228 us for the earlier layout that folded each block's absmax in LDS.
#ifndef ZPP_QGZ_GROUP_MIN_FILL
#define ZPP_QGZ_GROUP_MIN_FILL 75
#endif
#ifndef ZPP_QGZ_MAX_GRID
#define ZPP_QGZ_MAX_GRID (1u << 30)
#endif

namespace zpp {
namespace {

constexpr int kQgzThreads = ZPP_QGZ_THREADS;

struct I4Quant {
    float scale, pre, inv;
    bool zero, tiny;
};

__device__ __forceinline__ I4Quant i4_params(uint32_t absbits) {
    I4Quant q;
    const float a = __uint_as_float(absbits);
    q.tiny = a < 0x1p-100f;
    q.pre = q.tiny ? 0x1p64f : 1.0f;
    q.inv = 7.0f / (a * q.pre);
    if (absbits >= 0x7F800000u) {
        q.scale = __uint_as_float(kScaleNaNBits);
        q.zero = true;
    } else if (absbits == 0u) {
        q.scale = 0.0f;
        q.zero = true;
    } else {
        q.scale = a / 7.0f;
        q.zero = false;
    }
    return q;
}

// 4 values -> 4 int4 codes packed little-endian in 16 bits.  No clamp is
// needed: |x * inv| rounds to at most 7 (1 + 2^-24)^2 < 7.5.
__device__ __forceinline__ uint32_t i4_half(const f32x4 &x, const I4Quant &q) {
#pragma clang fp contract(off)
    uint32_t b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float xe = q.tiny ? x[e] * q.pre : x[e];
        b[e] = code_bits(xe * q.inv);
    }
    // low bytes side by side, then low nibbles: bytes 0 and 2 of t hold
    // (c0 | c1 << 4) and (c2 | c3 << 4)
    const uint32_t w = pack_low_bytes(b[0], b[1], b[2], b[3]) & 0x0F0F0F0Fu;
    const uint32_t t = w | (w >> 4);
    const uint32_t packed = __builtin_amdgcn_perm(0u, t, 0x0c0c0200u);
    return q.zero ? 0u : packed;
}

__device__ __forceinline__ uint32_t abs_bits_max4(const f32x4 &v) {
    return max(max(__float_as_uint(v.x) & 0x7FFFFFFFu, __float_as_uint(v.y) & 0x7FFFFFFFu),
               max(__float_as_uint(v.z) & 0x7FFFFFFFu, __float_as_uint(v.w) & 0x7FFFFFFFu));
}

// A lane holds groups of 4 consecutive values; group t of lane l in a wave's
// tile starts at 256 t + 4 l, so every load instruction of a wave reads 1 KiB
// and every code store writes 128 contiguous bytes.  A block of B values
// spans L = min(B/4, 64) lanes and G = max(1, B/256) groups per lane; a
// wave covers C = max(B, 256) values per tile and keeps U tiles in flight.
// Where the codes and scale of one source go in a receive buffer of P
// sources interleaved block by block (block k of B elements: source q's B/2
// code bytes at (k P + q) B/2, its scale at k P + q); P = 1, q = 0 is the
// plain layout (byte i / 2, scale k).
__device__ __forceinline__ size_t i4_out_byte(size_t i, uint32_t shift, uint32_t q, uint32_t P) {
    return (((i >> shift) * P + q) << (shift - 1)) + ((i & (((size_t)1 << shift) - 1)) >> 1);
}

// The same for element i of block k of any block size B.
__device__ __forceinline__ size_t i4_out_byte_any(size_t i, size_t k, uint32_t B, uint32_t q,
                                                  uint32_t P) {
    return (k * P + q) * (B / 2) + ((i - k * B) >> 1);
}

// One wave's U tiles from element `base` on, `rest` elements of them inside the
// array (WHOLE: all of them).
template <int B, int U, bool WHOLE>
__device__ __forceinline__ void quant_i4_tiles(const float *__restrict__ src, size_t base,
                                               uint32_t rest, uint8_t *__restrict__ codes,
                                               float *__restrict__ scales, uint32_t q_src,
                                               uint32_t num_src) {
    constexpr uint32_t kShift = __builtin_ctz(B);
    constexpr int C = B > 256 ? B : 256;
    constexpr int G = C / 256;
    constexpr int L = B < 256 ? B / 4 : kWave;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    src += base;
    f32x4 x[U][G];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t i = u * C + g * 256 + lane * 4;
            if (WHOLE || i + 4 <= rest) {
                x[u][g] = ld_nt_at<f32x4, 4>(src + i);
            } else {
                float h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    h[e] = i + e < rest ? src[i + e] : 0.0f;
                x[u][g] = f32x4{h[0], h[1], h[2], h[3]};
            }
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint32_t mx = 0;
#pragma unroll
        for (int g = 0; g < G; ++g)
            mx = max(mx, abs_bits_max4(x[u][g]));
#pragma unroll
        for (int off = L / 2; off >= 1; off >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        const I4Quant q = i4_params(mx);
        const auto store = [&](int g) {
            const uint32_t i = u * C + g * 256 + lane * 4;
            const uint32_t h = i4_half(x[u][g], q);
            const size_t byte0 = i4_out_byte(base + i, kShift, q_src, num_src);
            // the second byte holds elements i + 2 and i + 3
            if (WHOLE || i + 2 < rest)
                st_nt_at<uint16_t, 1>(codes + byte0, (uint16_t)h);
            else if (i < rest)
                codes[byte0] = (uint8_t)h;
        };
        // no loop over a single group: its store would be hoisted out of it as
        // a plain, temporal one
        if constexpr (G == 1) {
            store(0);
        } else {
#pragma unroll
            for (int g = 0; g < G; ++g)
                store(g);
        }
        if (lane % L == 0 && (WHOLE || u * C + lane * 4 < rest))
            scales[((base + u * C + lane * 4) / B) * num_src + q_src] = q.scale;
    }
}

template <int B, int U>
__global__ __launch_bounds__(kQgzThreads) void quant_i4_kernel(
    const float *__restrict__ src, uint8_t *__restrict__ codes, float *__restrict__ scales,
    uint32_t q_src, uint32_t num_src, TileSpan tiles) {
    constexpr uint32_t C = (B > 256 ? B : 256) * U;
    constexpr int kWaves = kQgzThreads / kWave;
    const uint32_t t =
        blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const size_t base = (tiles.first + t) * C;
    if (__builtin_expect(t < tiles.whole, 1))
        quant_i4_tiles<B, U, true>(src, base, C, codes, scales, q_src, num_src);
    else if (t == tiles.whole && tiles.tail)
        quant_i4_tiles<B, U, false>(src, base, tiles.tail, codes, scales, q_src, num_src);
}

// Vector path for a block B = 64 b that is not a power of two, lane-group
// layout (zpp_chunk.h): each block owns an aligned group of G lanes, lane r
// of the group holding the block's groups of 4 values v G + r for v < S
// (groups past the block's end stay empty).  The block absmax is a
// reduction over the group's G lanes with cross-lane xor shuffles and every
// lane derives the block's parameters itself, as in the power-of-two
// kernel: no LDS, no atomics and no barrier.  Workgroups whose blocks all
// lie inside the array load each group with one predicated load; only the
// last one checks every element.
template <int G, int S>
__global__ __launch_bounds__(kQgzThreads) void quant_i4_grp_kernel(
    const float *__restrict__ src, size_t n, uint32_t B, uint8_t *__restrict__ codes,
    float *__restrict__ scales, uint32_t q_src, uint32_t num_src) {
    constexpr int kBlocksPerWave = kWave / G;
    constexpr int kBlocksPerGroup = kBlocksPerWave * (kQgzThreads / kWave);
    const uint32_t gpb = B / 4;
    const size_t nblocks = (n + B - 1) / B;
    const int lane = threadIdx.x & (kWave - 1);
    const int li = lane % G;
    const size_t kw = (size_t)(threadIdx.x / kWave) * kBlocksPerWave + lane / G;
    for (size_t g0 = (size_t)blockIdx.x * kBlocksPerGroup; g0 < nblocks;
         g0 += (size_t)gridDim.x * kBlocksPerGroup) {
        const size_t k = g0 + kw;
        const bool valid = k < nblocks;
        const bool whole = (g0 + kBlocksPerGroup) * B <= n;  // uniform
        f32x4 x[S];
        if (whole) {
#pragma unroll
            for (int v = 0; v < S; ++v) {
                x[v] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                const uint32_t j = (uint32_t)(v * G + li);
                if (j < gpb)
                    x[v] = ld_nt_at<f32x4, 4>(src + k * B + (size_t)j * 4);
            }
        } else {
#pragma unroll
            for (int v = 0; v < S; ++v) {
                x[v] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                const uint32_t j = (uint32_t)(v * G + li);
                const size_t i = k * B + (size_t)j * 4;
                if (valid && j < gpb) {
                    if (i + 4 <= n) {
                        x[v] = ld_nt_at<f32x4, 4>(src + i);
                    } else if (i < n) {
                        float h[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            h[e] = (i + e < n) ? src[i + e] : 0.0f;
                        x[v] = f32x4{h[0], h[1], h[2], h[3]};
                    }
                }
            }
        }
        uint32_t mx = 0;
#pragma unroll
        for (int v = 0; v < S; ++v)
            mx = max(mx, abs_bits_max4(x[v]));
#pragma unroll
        for (int off = G / 2; off >= 1; off >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        const I4Quant q = i4_params(mx);
#pragma unroll
        for (int v = 0; v < S; ++v) {
            const uint32_t j = (uint32_t)(v * G + li);
            const size_t i = k * B + (size_t)j * 4;
            if (!valid || j >= gpb || i >= n)
                continue;
            const uint32_t h = i4_half(x[v], q);
            const size_t byte0 = i4_out_byte_any(i, k, B, q_src, num_src);
            // the second byte holds elements i + 2 and i + 3
            if (i + 2 < n)
                st_nt_at<uint16_t, 1>(codes + byte0, (uint16_t)h);
            else
                codes[byte0] = (uint8_t)h;
        }
        if (valid && li == 0)
            scales[k * num_src + q_src] = q.scale;
    }
}

// The dequant-reduce, from either gradient source of zpp_i4grad.h: a lane
// holds G groups of 4 consecutive elements at 256 g + 4 l of its wave's tile,
// so each source is read as 128-byte contiguous wave loads (2 bytes per lane)
// and every group is stored as one float4 (1 KiB contiguous per wave store).
// From separate arrays workgroups are renumbered in runs per XCD
// (kSeparateXcdRun), so that the tiles sharing a line of a source's scales
// read it through one L2.
template <class GS> constexpr size_t reduce_xcd_run() { return 0; }
template <> constexpr size_t reduce_xcd_run<I4Grad>() { return kSeparateXcdRun; }

template <class GS, int G, bool MANY>
__global__ __launch_bounds__(kQgzThreads) void reduce_gs_kernel(GS gs, float *__restrict__ out,
                                                               TileSpan tiles) {
    constexpr int kWaves = kQgzThreads / kWave;
    constexpr size_t C = 256 * G;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, tiles, reduce_xcd_run<GS>()) * kWaves + wave;
    const size_t base = (tiles.first + t) * C;
    f32x4 r[G];
    if (__builtin_expect(t < tiles.whole, 1)) {
        grad_tile<true, MANY>(r, gs, base, lane, C);
#pragma unroll
        for (int g = 0; g < G; ++g)
            store4<true>(out + base, g * 256 + lane * 4, C, r[g]);
    } else if (t == tiles.whole && tiles.tail) {
        grad_tile<false, MANY>(r, gs, base, lane, tiles.tail);
#pragma unroll
        for (int g = 0; g < G; ++g)
            store4<false>(out + base, g * 256 + lane * 4, tiles.tail, r[g]);
    }
}

template <int G, bool MANY, class GS>
void launch_reduce_gs(const GS &gs, size_t n, float *out, bool on_lines, hipStream_t stream) {
    for_tiles(n, 256 * G, kQgzThreads / kWave, kQgzThreads, on_lines,
              [&](const TileSpan &tiles, unsigned grid) {
                  hipLaunchKernelGGL((reduce_gs_kernel<GS, G, MANY>), dim3(grid),
                                     dim3(kQgzThreads), 0, stream, gs, out, tiles);
              });
}

// MANY sources: two groups per lane stream better (13.1 M elements of 16
// separate copies: 32.9 against 35.4 us, 50 M: 117 against 127), one puts a
// short array on more waves (500,000 elements: 3.1 against 4.1 us): two from
// the length that gives every CU its 32 waves.  Fewer sources keep two.
template <class GS>
hipError_t launch_reduce(const GS &gs, size_t n, float *out, bool on_lines, hipStream_t stream) {
    if (!many_sources(gs.num_src, gs.block.block))
        launch_reduce_gs<2, false>(gs, n, out, on_lines, stream);
    else if (n >= (size_t)512 * 32 * kCUs)
        launch_reduce_gs<2, true>(gs, n, out, on_lines, stream);
    else
        launch_reduce_gs<1, true>(gs, n, out, on_lines, stream);
    return hipGetLastError();
}

// Workgroups per CU.  One tile of a large block per wave into a sender's slots,
// whose scales land between the other senders', streams better with fewer
// resident once the array is long (8 senders, uncapped -> capped: 1024 at 60 M
// / 100 M / 203 M elements 50.6 -> 48.1, 86.9 -> 79.8, 182 -> 166 us; 4096, at
// 2, 53.6 -> 50.8, 88.8 -> 83.1, 180 -> 167; 2048, at 2 and with two tiles per
// wave, 48.4 -> 48.4, 81.6 -> 77.6, 170 -> 156; with one at 4, 166); blocks up
// to 512 gain nothing.
template <int B>
int quant_i4_residency(size_t n, uint32_t num_src) {
    if (B < 1024 || num_src == 1 || n < (size_t)48 << 20)
        return 0;
    return B == 1024 ? 4 : 2;
}

template <int B, int U>
void launch_quant_i4_u(const float *src, size_t n, uint8_t *codes, float *scales, uint32_t q_src,
                       uint32_t num_src, hipStream_t stream) {
    const size_t lds = residency_lds(quant_i4_residency<B>(n, num_src));
    for_tiles(n, (B > 256 ? B : 256) * U, kQgzThreads / kWave, kQgzThreads, true,
              [&](const TileSpan &tiles, unsigned grid) {
                  hipLaunchKernelGGL((quant_i4_kernel<B, U>), dim3(grid), dim3(kQgzThreads), lds,
                                     stream, src, codes, scales, q_src, num_src, tiles);
              });
}

// Tiles of max(B, 256) elements a wave keeps in flight.  Blocks of 512 and
// more fill a lane's registers with one (four took 24.1 / 24.2 / 36.7 us at
// blocks of 512 / 1024 / 4096 and 25.9 M elements, one 19.9 / 20.2 / 21.4;
// 203 M: 151 / 152 / 219, and 143 / 148 / 162).  Up to 256 four stream best
// over long arrays (203 M: 147 us, 160 with two), two put a short one on more
// waves (i4_two_tiles, zpp_chunk.h).
template <int B>
void launch_quant_i4_b(const float *src, size_t n, uint8_t *codes, float *scales,
                       uint32_t q_src, uint32_t num_src, hipStream_t stream) {
    if constexpr (B == 2048) {
        if (quant_i4_residency<B>(n, num_src) != 0)
            return launch_quant_i4_u<B, 2>(src, n, codes, scales, q_src, num_src, stream);
    }
    if constexpr (B > 256)
        launch_quant_i4_u<B, 1>(src, n, codes, scales, q_src, num_src, stream);
    else if (i4_two_tiles(B, num_src, n))
        launch_quant_i4_u<B, 2>(src, n, codes, scales, q_src, num_src, stream);
    else
        launch_quant_i4_u<B, 4>(src, n, codes, scales, q_src, num_src, stream);
}

template <int G, int S>
void launch_quant_i4_grp(const float *src, size_t n, uint32_t block, uint8_t *codes,
                         float *scales, uint32_t q_src, uint32_t num_src, hipStream_t stream) {
    constexpr size_t kBlocksPerGroup = (kWave / G) * (kQgzThreads / kWave);
    const size_t nblocks = (n + block - 1) / block;
    const size_t need = (nblocks + kBlocksPerGroup - 1) / kBlocksPerGroup;
    const unsigned grid = (unsigned)(need < ZPP_QGZ_MAX_GRID ? need : ZPP_QGZ_MAX_GRID);
    hipLaunchKernelGGL((quant_i4_grp_kernel<G, S>), dim3(grid), dim3(kQgzThreads), 0, stream,
                       src, n, block, codes, scales, q_src, num_src);
}

template <int S>
void launch_quant_i4_grp_g(uint32_t G, const float *src, size_t n, uint32_t block,
                           uint8_t *codes, float *scales, uint32_t q_src, uint32_t num_src,
                           hipStream_t stream) {
    switch (G) {
    case 16: launch_quant_i4_grp<16, S>(src, n, block, codes, scales, q_src, num_src, stream); break;
    case 32: launch_quant_i4_grp<32, S>(src, n, block, codes, scales, q_src, num_src, stream); break;
    default: launch_quant_i4_grp<64, S>(src, n, block, codes, scales, q_src, num_src, stream); break;
    }
}

}  // namespace

hipError_t launch_quantize_i4_il(const float *src, size_t n, uint32_t block, uint32_t source,
                                 uint32_t num_src, uint8_t *codes, float *scales,
                                 hipStream_t stream) {
    switch (block) {
    case 64: launch_quant_i4_b<64>(src, n, codes, scales, source, num_src, stream); break;
    case 128: launch_quant_i4_b<128>(src, n, codes, scales, source, num_src, stream); break;
    case 256: launch_quant_i4_b<256>(src, n, codes, scales, source, num_src, stream); break;
    case 512: launch_quant_i4_b<512>(src, n, codes, scales, source, num_src, stream); break;
    case 1024: launch_quant_i4_b<1024>(src, n, codes, scales, source, num_src, stream); break;
    case 2048: launch_quant_i4_b<2048>(src, n, codes, scales, source, num_src, stream); break;
    case 4096: launch_quant_i4_b<4096>(src, n, codes, scales, source, num_src, stream); break;
    default: {
        const GroupShape sh = group_shape(block / 4, 16, ZPP_QGZ_GROUP_MIN_FILL, 3);
        if (sh.S <= 4)
            launch_quant_i4_grp_g<4>(sh.G, src, n, block, codes, scales, source, num_src,
                                     stream);
        else if (sh.S <= 8)
            launch_quant_i4_grp_g<8>(sh.G, src, n, block, codes, scales, source, num_src,
                                     stream);
        else
            launch_quant_i4_grp_g<16>(sh.G, src, n, block, codes, scales, source, num_src,
                                      stream);
    }
    }
    return hipGetLastError();
}

hipError_t launch_quantize_i4(const float *src, size_t n, uint32_t block, uint8_t *codes,
                              float *scales, hipStream_t stream) {
    return launch_quantize_i4_il(src, n, block, 0, 1, codes, scales, stream);
}

hipError_t launch_dequant_reduce_i4(const uint8_t *const *src_codes,
                                    const float *const *src_scales, uint32_t num_src, size_t n,
                                    uint32_t block, float scale_out, float *out,
                                    bool on_lines, hipStream_t stream) {
    return launch_reduce(make_i4grad(src_codes, src_scales, num_src, block, scale_out), n, out,
                         on_lines, stream);
}

hipError_t launch_dequant_reduce_i4_il(const uint8_t *codes, const float *scales, uint32_t num_src,
                                       size_t n, uint32_t block, float scale_out, float *out,
                                       bool on_lines, hipStream_t stream) {
    return launch_reduce(make_i4grad_il(codes, scales, num_src, block, scale_out), n, out,
                         on_lines, stream);
}

}  // namespace zpp
