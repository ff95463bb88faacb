// Fused partition step: the Adam update of the rank's partition, its bf16
// primary, the hpZ secondary copy and the qwZ int8 quantization of that copy,
// in one pass over HBM (optimizer.step() of Algorithm 1 followed, for the
// same weights, by the secondary copy of the forward loop and the qwZ
// quantization that precedes the gather).
//
// Per element: 16 B read (p, m, v, g); 12 B + 2 B + 2 B + 1 B written (p, m,
// v, primary, secondary, code) plus 4 B per block of scale: 33.016 B at block
// 256, against 30 + 4 + 3.016 = 37.016 B for the three separate kernels,
// which re-read the primary and the secondary from HBM.  The results are
// those of the three separate steps, bit for bit, because the quantization
// reads the same bf16 values the primary holds.
//
// One wave per chunk of C = max(B, 256) consecutive elements: lane l holds
// the 4 elements [chunk + 256 w + 4 l, +4) for w < C / 256.  The bf16 of the
// updated weights stays in registers (two per 4 elements) until the block's
// absmax is known; a 256-block is exactly one wave, so its absmax is a
// six-step cross-lane reduction.  Blocks of 64, 128, 256 and 512 take this
// kernel.  Any other block takes a workgroup per block (fused_wide_kernel)
// where that is faster (wide_block, zpp_chunk.h), or two passes: the same kernel
// with the 256-element chunks and no quantization (p, m, v, primary, secondary:
// 32 B per element), then the int8 quantizer over the primary it wrote (3 B +
// 4/B B), in stream order.  Over a long array the 2 extra bytes per element cost
// less than holding a larger block's values in a wave: at the Llama-2-13B
// partition the two passes took 1094-1104 us at blocks of 192 to 4096, the
// one-pass layouts 1127-1186 us (one wave per chunk of whole blocks, several
// blocks per wave with the maxima in LDS, or workgroups of up to 16 waves
// with one float4 group per thread and a barrier per block), all but 512
// (1073 against 1095 us one pass); the single pass of the qgZ receive took
// 1112-1117 against 1245-1460 us.
// Residency is capped at ZPP_FUSED_RESIDENCY workgroups per CU, as for the optimizer step: 1031-1046 us with 11 resident
// at the Llama-2-13B partition (9-18 within 1%), 1127-1145 us uncapped.  With
// the qgZ receive in place of the fp32 gradient (8 int4 sources) the cap is
// ZPP_FUSED_RECV_RESIDENCY: 1111 us with 12, 1118 with 14, 1150 with 11, 1216
// with 10, 1142 uncapped.  From one interleaved receive buffer
// (ZPP_FUSED_RECV_IL_RESIDENCY): 1054 us with 14, 1062 with 16, 1075 with 11,
// 1097 uncapped, against 1096 us from separate arrays in the same run.
#include <type_traits>

#include "zpp_adam.h"
#include "zpp_chunk.h"
#include "zpp_device.h"
#include "zpp_i4grad.h"
#include "zpp_launch.h"
#include "zpp_quant.h"

#ifndef ZPP_FUSED_RESIDENCY
#define ZPP_FUSED_RESIDENCY 11
#endif
#ifndef ZPP_FUSED_RECV_RESIDENCY
#define ZPP_FUSED_RECV_RESIDENCY 12
#endif
#ifndef ZPP_FUSED_RECV_IL_RESIDENCY
#define ZPP_FUSED_RECV_IL_RESIDENCY 14
#endif
namespace zpp {
namespace {

struct FusedArgs {
    float *p, *m, *v;
    uint16_t *primary;
    uint16_t *secondary;  // may be null: no bf16 secondary copy is kept
    int8_t *codes;
    float *scales;
    size_t n;
    AdamConsts c;
};

template <class GS> constexpr Gradient gradient();
template <> constexpr Gradient gradient<F32Grad>() { return Gradient::kF32; }
template <> constexpr Gradient gradient<I4Grad>() { return Gradient::kCopies; }
template <> constexpr Gradient gradient<I4GradIl>() { return Gradient::kInterleaved; }
inline uint32_t num_sources(const F32Grad &) { return 0; }
template <class GS> uint32_t num_sources(const GS &gs) { return gs.num_src; }

// Runs of consecutive workgroups per XCD: grouped for the qgZ receive from
// separate arrays (zpp_i4grad.h), plain otherwise.
template <class GS> constexpr size_t fused_xcd_run() { return 0; }
template <> constexpr size_t fused_xcd_run<I4Grad>() { return kSeparateXcdRun; }

// One chunk of C consecutive elements from `base` on, `rest` of which lie
// inside the arrays.  WHOLE: all of them; otherwise (the launch's last,
// partial chunk) the absent elements hold bf16 zero, which no absmax can see.
template <bool ADAMW, int B, bool QUANT, bool WHOLE, bool MANY, class GS>
__device__ __forceinline__ void fused_chunk(const FusedArgs &a, const GS &gs, size_t base,
                                            uint32_t rest) {
    constexpr int C = B > 256 ? B : 256;  // elements per chunk (one wave)
    constexpr int W = C / 256;            // float4 groups per lane
    static_assert(W <= 2, "blocks of 64 to 512");
    constexpr int L = B < 256 ? B / 4 : kWave;  // lanes per quant block
    const uint32_t lane = threadIdx.x;
    f32x4 P[W], M[W], V[W], G[W];
    u32x2 pk[W];
    u16x2 m2 = {0, 0};
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t i = w * 256 + lane * 4;
        P[w] = load4<WHOLE>(a.p + base, i, rest);
        M[w] = load4<WHOLE>(a.m + base, i, rest);
        V[w] = load4<WHOLE>(a.v + base, i, rest);
    }
    grad_tile<WHOLE, MANY>(G, gs, base, lane, rest);
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t i = w * 256 + lane * 4;
        adam_update4<ADAMW>(P[w], M[w], V[w], G[w], a.c);
        store4<WHOLE>(a.p + base, i, rest, P[w]);
        store4<WHOLE>(a.m + base, i, rest, M[w]);
        store4<WHOLE>(a.v + base, i, rest, V[w]);
        pk[w] = u32x2{pack_bf16x2(P[w].x, P[w].y), pack_bf16x2(P[w].z, P[w].w)};
        if constexpr (!WHOLE) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e >= rest)
                    pk[w][e / 2] &= e % 2 ? 0x0000FFFFu : 0xFFFF0000u;
        }
        store4_bf16<WHOLE>(a.primary + base, i, rest, pk[w]);
        if (a.secondary)
            store4_bf16<WHOLE>(a.secondary + base, i, rest, pk[w]);
        m2 = __builtin_elementwise_max(
            m2, __builtin_elementwise_max(absbits2(pk[w].x), absbits2(pk[w].y)));
    }
    if constexpr (QUANT) {
        uint32_t mx = max((uint32_t)m2.x, (uint32_t)m2.y);
#pragma unroll
        for (int off = L / 2; off >= 1; off >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
        const BlockQuant q = block_params(mx);
        // no loop: its one store would be hoisted out of it as a plain,
        // temporal one
        store4_i8<WHOLE>(a.codes + base, lane * 4, rest, quant_word(pk[0].x, pk[0].y, q));
        if constexpr (W == 2)
            store4_i8<WHOLE>(a.codes + base, 256 + lane * 4, rest,
                             quant_word(pk[1].x, pk[1].y, q));
        // the first lane of each quant block writes its scale
        if (lane % L == 0 && lane * 4 < rest)
            a.scales[base / B + lane * 4 / B] = q.scale;
    }
}

// The gradient comes from `gs`: the fp32 array of the partition step
// (F32Grad), or the int4 copies of the qgZ receive (I4Grad, zpp_i4grad.h).
template <bool ADAMW, int B, class GS, bool QUANT, bool MANY>
__global__ __launch_bounds__(kWave) void fused_kernel(FusedArgs a, GS gs, TileSpan chunks) {
    constexpr uint32_t C = B > 256 ? B : 256;
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, chunks, fused_xcd_run<GS>());
    const size_t base = (chunks.first + t) * C;
    if (__builtin_expect(t < chunks.whole, 1))
        fused_chunk<ADAMW, B, QUANT, true, MANY>(a, gs, base, C);
    else
        fused_chunk<ADAMW, B, QUANT, false, MANY>(a, gs, base, chunks.tail);
}

// The fused step with one quant block per workgroup, for blocks other than 64,
// 128, 256 and 512: ceil(B / 256) waves, one float4 group per lane (the lanes past a
// block that is no multiple of 256 stay idle), the waves' maxima exchanged in
// LDS.  The block's values stay in registers, so the primary is not read back
// and there is one launch instead of two.
template <bool ADAMW, bool WHOLE, bool MANY, class GS>
__device__ __forceinline__ void fused_wide_block(const FusedArgs &a, const GS &gs, size_t base,
                                                 uint32_t rest, size_t k) {
    __shared__ uint32_t wave_mx[16];
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t waves = blockDim.x / kWave;
    const uint32_t i = threadIdx.x * 4;
    const size_t wb = base + wave * 256;
    const bool some = WHOLE ? i < rest : wave * 256 < rest;
    u32x2 pk = {0u, 0u};
    if (some) {
        f32x4 P = load4<WHOLE>(a.p + base, i, rest), M = load4<WHOLE>(a.m + base, i, rest),
              V = load4<WHOLE>(a.v + base, i, rest), G[1];
        grad_tile<WHOLE, MANY>(G, gs, wb, lane, rest - wave * 256);
        adam_update4<ADAMW>(P, M, V, G[0], a.c);
        pk = u32x2{pack_bf16x2(P.x, P.y), pack_bf16x2(P.z, P.w)};
        if constexpr (!WHOLE) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e >= rest)
                    pk[e / 2] &= e % 2 ? 0x0000FFFFu : 0xFFFF0000u;
        }
        store4<WHOLE>(a.p + base, i, rest, P);
        store4<WHOLE>(a.m + base, i, rest, M);
        store4<WHOLE>(a.v + base, i, rest, V);
        store4_bf16<WHOLE>(a.primary + base, i, rest, pk);
        if (a.secondary)
            store4_bf16<WHOLE>(a.secondary + base, i, rest, pk);
    }
    const u16x2 m2 = __builtin_elementwise_max(absbits2(pk.x), absbits2(pk.y));
    uint32_t mx = max((uint32_t)m2.x, (uint32_t)m2.y);
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1)
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
    if (lane == 0)
        wave_mx[wave] = mx;
    // the waves meet once their maxima are in LDS; their stores to memory
    // need not have finished, so this is no __syncthreads()
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    mx = lane < waves ? wave_mx[lane % 16] : 0u;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
    mx = __builtin_amdgcn_readfirstlane(mx);
    const BlockQuant q = block_params(mx);
    if (some)
        store4_i8<WHOLE>(a.codes + base, i, rest, quant_word(pk.x, pk.y, q));
    if (threadIdx.x == 0)
        a.scales[k] = q.scale;
}

template <bool ADAMW, bool MANY, class GS>
__global__ __launch_bounds__(1024) void fused_wide_kernel(FusedArgs a, GS gs, uint32_t B,
                                                          TileSpan blocks) {
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, blocks, fused_xcd_run<GS>() / 4);
    const size_t k = blocks.first + t;
    if (__builtin_expect(t < blocks.whole, 1))
        fused_wide_block<ADAMW, true, MANY>(a, gs, k * B, B, k);
    else
        fused_wide_block<ADAMW, false, MANY>(a, gs, k * B, blocks.tail, k);
}

// Workgroups per CU: the step's three or four times four waves (1024 at 45 M:
// 236 us with 3, 249 with 4, 256 left to the hardware; the receive at 50 M 278
// / 271 / 279), but short launches and many sources are left to the hardware
// (1024 at 1 M elements: 6.9 us against 7.6 with 3).
template <class GS>
int wide_residency(const GS &gs, size_t n) {
    if (n <= kWideShort / 2)
        return 0;
    if constexpr (std::is_same_v<GS, F32Grad>)
        return 3;
    else
        return gs.num_src >= kManySources ? 0 : 4;
}

template <bool MANY, class GS>
void launch_wide(const FusedArgs &a, const GS &gs, uint32_t block, bool on_lines,
                 hipStream_t stream) {
    const uint32_t threads = (block / 4 + kWave - 1) / kWave * kWave;
    // beyond half of kWideShort a block of fewer waves would be capped too low
    const int per_cu = threads / kWave >= 4 ? wide_residency(gs, a.n) : 0;
    // the maxima have a granule of their own
    const size_t lds = per_cu ? residency_lds(per_cu) - kLdsGranule : 0;
    for_tiles(a.n, block, 1, threads, on_lines, [&](const TileSpan &blocks, unsigned grid) {
        if (a.c.adamw)
            hipLaunchKernelGGL((fused_wide_kernel<true, MANY, GS>), dim3(grid), dim3(threads),
                               lds, stream, a, gs, block, blocks);
        else
            hipLaunchKernelGGL((fused_wide_kernel<false, MANY, GS>), dim3(grid), dim3(threads),
                               lds, stream, a, gs, block, blocks);
    });
}

// Workgroups per CU for each gradient source.
template <class GS> constexpr int fused_residency();
template <> constexpr int fused_residency<F32Grad>() { return ZPP_FUSED_RESIDENCY; }
template <> constexpr int fused_residency<I4Grad>() { return ZPP_FUSED_RECV_RESIDENCY; }
template <> constexpr int fused_residency<I4GradIl>() { return ZPP_FUSED_RECV_IL_RESIDENCY; }

template <int B, bool QUANT, bool MANY, class GS>
void launch_fused_chunks(const FusedArgs &a, const GS &gs, int residency, bool on_lines,
                         hipStream_t stream) {
    constexpr uint32_t C = B > 256 ? B : 256;
    const size_t lds = launch_lds(residency, a.n / C);
    for_tiles(a.n, C, 1, kWave, on_lines, [&](const TileSpan &chunks, unsigned grid) {
        if (a.c.adamw)
            hipLaunchKernelGGL((fused_kernel<true, B, GS, QUANT, MANY>), dim3(grid), dim3(kWave),
                               lds, stream, a, gs, chunks);
        else
            hipLaunchKernelGGL((fused_kernel<false, B, GS, QUANT, MANY>), dim3(grid), dim3(kWave),
                               lds, stream, a, gs, chunks);
    });
}

template <int B, bool QUANT = true, class GS>
void launch_fused_b(const FusedArgs &a, const GS &gs, bool on_lines, hipStream_t stream) {
    int residency = fused_residency<GS>();
    if constexpr (!QUANT)
        residency = copies_residency(gradient<GS>(), residency);
    if constexpr (!std::is_same_v<GS, F32Grad>) {
        residency = receive_residency(gradient<GS>(), gs.num_src, gs.block.block, a.n, QUANT,
                                      residency);
        if (many_sources(gs.num_src, gs.block.block))
            return launch_fused_chunks<B, QUANT, true>(a, gs, residency, on_lines, stream);
    }
    launch_fused_chunks<B, QUANT, false>(a, gs, residency, on_lines, stream);
}

template <class GS>
hipError_t launch_fused_gs(const FusedArgs &a, const GS &gs, uint32_t block, bool on_lines,
                           hipStream_t stream) {
    switch (block) {
    case 64: launch_fused_b<64>(a, gs, on_lines, stream); break;
    case 128: launch_fused_b<128>(a, gs, on_lines, stream); break;
    case 256: launch_fused_b<256>(a, gs, on_lines, stream); break;
    case 512: launch_fused_b<512>(a, gs, on_lines, stream); break;
    default: {
        if (wide_block(gradient<GS>(), num_sources(gs), block, a.n)) {
            if constexpr (!std::is_same_v<GS, F32Grad>) {
                // a wave's 256 elements lie in one int4 block
                if (block % 256 == 0 && many_sources(gs.num_src, gs.block.block)) {
                    launch_wide<true>(a, gs, block, on_lines, stream);
                    return hipGetLastError();
                }
            }
            launch_wide<false>(a, gs, block, on_lines, stream);
            return hipGetLastError();
        }
        // the step and its copies in one pass, then the quantization of
        // the primary it wrote (stream order)
        launch_fused_b<256, false>(a, gs, on_lines, stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        return launch_quantize(a.primary, a.n, block, a.codes, a.scales, stream);
    }
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused(float *p, float *m, float *v, const float *g, uint16_t *primary,
                        uint16_t *secondary, int8_t *codes, float *scales, size_t n,
                        uint32_t block, const AdamConsts &c, bool on_lines, hipStream_t stream) {
    const FusedArgs a{p, m, v, primary, secondary, codes, scales, n, c};
    return launch_fused_gs(a, F32Grad{g}, block, on_lines, stream);
}

hipError_t launch_fused_receive(float *p, float *m, float *v, const uint8_t *const *src_codes,
                                const float *const *src_scales, uint32_t num_src,
                                uint32_t grad_block, float scale_out, uint16_t *primary,
                                uint16_t *secondary, int8_t *codes, float *scales, size_t n,
                                uint32_t block, const AdamConsts &c, bool on_lines,
                                hipStream_t stream) {
    const FusedArgs a{p, m, v, primary, secondary, codes, scales, n, c};
    return launch_fused_gs(a, make_i4grad(src_codes, src_scales, num_src, grad_block, scale_out),
                           block, on_lines, stream);
}

hipError_t launch_fused_receive_il(float *p, float *m, float *v, const uint8_t *src_codes,
                                   const float *src_scales, uint32_t num_src, uint32_t grad_block,
                                   float scale_out, uint16_t *primary, uint16_t *secondary,
                                   int8_t *codes, float *scales, size_t n, uint32_t block,
                                   const AdamConsts &c, bool on_lines, hipStream_t stream) {
    const FusedArgs a{p, m, v, primary, secondary, codes, scales, n, c};
    return launch_fused_gs(a, make_i4grad_il(src_codes, src_scales, num_src, grad_block, scale_out),
                           block, on_lines, stream);
}

}  // namespace zpp
