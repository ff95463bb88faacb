// qgZ receive fused into the partition step: the rank's optimizer step takes
// its gradient straight from the P int4 copies of its partition that the
// exchange replacing the ReduceScatter delivered (Background section: qgZ;
// Algorithm 1, backward loop, and the optimizer.step() closing it), instead
// of reading an fp32 gradient that a separate dequantize-and-reduce wrote.
//
// Per element: 12 B read (p, m, v) plus P (0.5 B + 4/B B) of codes and
// scales, 14 B written (p, m, v, bf16 primary): 30.125 B at P = 8 and block
// 256, against 8.125 + 30 B for the two kernels in sequence, which write the
// fp32 gradient and read it back.  The gradient is formed exactly as the
// dequantize-and-reduce forms it (acc = fma(code, scale, acc) over the
// sources in order from acc = 0, then one multiply by the output scale) and
// the update is the partition step's own, so the results are those of the
// two calls, bit for bit.
//
// Lane layout of the partition step: one wave per 256-element tile, lane l
// holds elements [256 t + 4 l, +4): one 16-byte access per state array, one
// 2-byte load of codes per source (a wave reads 128 contiguous bytes of each
// source) and one scale per source (zpp_i4grad.h: sources taken eight at a
// time, all eight in flight before their fma passes).  Residency is capped at
// ZPP_RECV_RESIDENCY workgroups per CU: at the Llama-2-13B partition with 8
// sources 994-1001 us with 11 (12: 995-999, 10: 1001-1008, 14: 1003-1011),
// 1027 us uncapped.  Scales loaded as wave-uniform scalar loads (possible for
// blocks of 256 or more) took 1112-1251 us: the scalar cache's latency is not
// hidden the way the vector loads' is.
//
// The same kernel reads the P copies from one interleaved receive buffer
// (I4GradIl, zpp_i4grad.h: a wave's codes of all sources within one
// contiguous run): 938 us with ZPP_RECV_IL_RESIDENCY = 11 (14: 949, 16: 955,
// uncapped 978) against 981 us from separate arrays in the same run.
#include <type_traits>

#include "zpp_adam.h"
#include "zpp_chunk.h"
#include "zpp_device.h"
#include "zpp_i4grad.h"
#include "zpp_launch.h"

#ifndef ZPP_RECV_RESIDENCY
#define ZPP_RECV_RESIDENCY 11
#endif
#ifndef ZPP_RECV_IL_RESIDENCY
#define ZPP_RECV_IL_RESIDENCY 11
#endif
namespace zpp {
namespace {

// The gradient comes from `src`: the P int4 copies as separate arrays
// (I4Grad) or interleaved in one receive buffer (I4GradIl, zpp_i4grad.h).
template <class GS>
struct RecvArgs {
    GS src;
    float *p, *m, *v;
    uint16_t *out;
    size_t n;
    AdamConsts c;
};

// Runs of consecutive workgroups per XCD: grouped for the separate arrays
// (zpp_i4grad.h), plain otherwise.
template <class GS> constexpr size_t recv_xcd_run() { return 0; }
template <> constexpr size_t recv_xcd_run<I4Grad>() { return kSeparateXcdRun; }

template <bool ADAMW, bool WHOLE, bool MANY, class GS>
__device__ __forceinline__ void recv_tile(const RecvArgs<GS> &a, size_t base, uint32_t rest) {
    const uint32_t i = threadIdx.x * 4;
    f32x4 P = load4<WHOLE>(a.p + base, i, rest);
    f32x4 M = load4<WHOLE>(a.m + base, i, rest);
    f32x4 V = load4<WHOLE>(a.v + base, i, rest);
    f32x4 G[1];
    grad_tile<WHOLE, MANY>(G, a.src, base, threadIdx.x, rest);
    adam_update4<ADAMW>(P, M, V, G[0], a.c);
    store4<WHOLE>(a.p + base, i, rest, P);
    store4<WHOLE>(a.m + base, i, rest, M);
    store4<WHOLE>(a.v + base, i, rest, V);
    store4_bf16<WHOLE>(a.out + base, i, rest,
                       u32x2{pack_bf16x2(P.x, P.y), pack_bf16x2(P.z, P.w)});
}

template <bool ADAMW, bool MANY, class GS>
__global__ __launch_bounds__(kWave) void recv_adam_kernel(RecvArgs<GS> a, TileSpan tiles) {
    const uint32_t t = tile_of(blockIdx.x, gridDim.x, tiles, recv_xcd_run<GS>());
    const size_t base = (tiles.first + t) * 256;
    if (__builtin_expect(t < tiles.whole, 1))
        recv_tile<ADAMW, true, MANY>(a, base, 256);
    else
        recv_tile<ADAMW, false, MANY>(a, base, tiles.tail);
}

template <bool MANY, class GS>
void launch_recv_tiles(const RecvArgs<GS> &a, int residency, bool on_lines, hipStream_t stream) {
    const size_t lds = launch_lds(residency, a.n / 256);
    for_tiles(a.n, 256, 1, kWave, on_lines, [&](const TileSpan &tiles, unsigned grid) {
        if (a.c.adamw)
            hipLaunchKernelGGL((recv_adam_kernel<true, MANY, GS>), dim3(grid), dim3(kWave), lds,
                               stream, a, tiles);
        else
            hipLaunchKernelGGL((recv_adam_kernel<false, MANY, GS>), dim3(grid), dim3(kWave), lds,
                               stream, a, tiles);
    });
}

template <class GS>
hipError_t launch_recv(const RecvArgs<GS> &a, int residency, bool on_lines, hipStream_t stream) {
    constexpr Gradient from =
        std::is_same_v<GS, I4Grad> ? Gradient::kCopies : Gradient::kInterleaved;
    residency = receive_residency(from, a.src.num_src, a.src.block.block, a.n, true, residency);
    if (many_sources(a.src.num_src, a.src.block.block))
        launch_recv_tiles<true>(a, residency, on_lines, stream);
    else
        launch_recv_tiles<false>(a, residency, on_lines, stream);
    return hipGetLastError();
}

}  // namespace

I4Grad make_i4grad(const uint8_t *const *src_codes, const float *const *src_scales,
                   uint32_t num_src, uint32_t block, float scale_out) {
    I4Grad s = {};
    for (uint32_t q = 0; q < num_src; ++q) {
        s.codes[q] = src_codes[q];
        s.scales[q] = src_scales[q];
    }
    s.num_src = num_src;
    s.block = make_block_div(block);
    s.scale_out = scale_out;
    return s;
}

hipError_t launch_receive_adam(float *p, float *m, float *v, const uint8_t *const *src_codes,
                               const float *const *src_scales, uint32_t num_src, uint32_t block,
                               float scale_out, uint16_t *out, size_t n, const AdamConsts &c,
                               bool on_lines, hipStream_t stream) {
    RecvArgs<I4Grad> a = {};
    a.src = make_i4grad(src_codes, src_scales, num_src, block, scale_out);
    a.p = p;
    a.m = m;
    a.v = v;
    a.out = out;
    a.n = n;
    a.c = c;
    return launch_recv(a, ZPP_RECV_RESIDENCY, on_lines, stream);
}

I4GradIl make_i4grad_il(const uint8_t *codes, const float *scales, uint32_t num_src,
                        uint32_t block, float scale_out) {
    I4GradIl s = {};
    s.codes = codes;
    s.scales = scales;
    s.num_src = num_src;
    s.block = make_block_div(block);
    s.scale_out = scale_out;
    return s;
}

hipError_t launch_receive_adam_il(float *p, float *m, float *v, const uint8_t *codes,
                                  const float *scales, uint32_t num_src, uint32_t block,
                                  float scale_out, uint16_t *out, size_t n, const AdamConsts &c,
                                  bool on_lines, hipStream_t stream) {
    RecvArgs<I4GradIl> a = {};
    a.src = make_i4grad_il(codes, scales, num_src, block, scale_out);
    a.p = p;
    a.m = m;
    a.v = v;
    a.out = out;
    a.n = n;
    a.c = c;
    return launch_recv(a, ZPP_RECV_IL_RESIDENCY, on_lines, stream);
}

}  // namespace zpp
