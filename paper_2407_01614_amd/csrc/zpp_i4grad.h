// The gradient that the qgZ receive delivers to the partition step: the sum,
// over the num_src int4 copies of the rank's partition (one from each sending
// rank, in rank order), of code * scale, accumulated with one fma per source
// from 0, then one multiply by the output scale (1/P for the data-parallel
// mean).  The dequantize-and-reduce kernel forms exactly this value and
// writes it; the kernels that take the receive into the optimizer step form
// it here, so that their results are bit for bit those of the separate calls.
#pragma once

#include "zpp_device.h"
#include "zpp_launch.h"
#include "zpp_quant.h"

namespace zpp {

// Workgroup numbering of the kernels that read the P copies from separate
// arrays (xcd_grouped in zpp_chunk.h): a 128-byte line of one source's
// scales serves 32 blocks, so 32 or more neighbouring tiles read it, and
// runs of this many consecutive workgroups per XCD let one L2 fetch it.  At
// the Llama-2-13B partition with 8 sources (median of 20 launches): the
// dequant-reduce 285 against 305 us, the receive step 990 against 1110, the
// single receive pass 1155 against 1235 (runs of 16 / 32 / 64 in between).
// The interleaved buffer keeps a block's scales of all sources in one
// 32-byte run, and the fused step has no shared lines: both were as fast or
// slower with grouping (the fused step 1079-1152 against 1046 us), so their
// kernels keep the plain numbering.
constexpr size_t kSeparateXcdRun = 128;

struct I4Grad {
    const uint8_t *codes[kMaxShards];  // packed int4, element 2i in the low nibble
    const float *scales[kMaxShards];   // one per block
    uint32_t num_src;
    BlockDiv block;
    float scale_out;
};

// The output scale, applied as its own rounded multiply: the separate calls
// store this product to memory before the update reads it, so it must not be
// contracted into an add of the update.
__device__ __forceinline__ float i4grad_scaled(float acc, float scale_out) {
#pragma clang fp contract(off)
    return acc * scale_out;
}

// The gradient of a lane's groups of four consecutive elements, group g at
// 256 g + 4 lane of a tile: one 2-byte code load and one scale per source and
// group.  N sources at a time, all their loads in flight before the fma
// passes, which keep the source order: eight, and what is left in one batch
// of that length.  No source carries a test: tested one by one, each load
// ended up in a branch of its own (the receive step at the Llama-2-13B
// partition 945 against 974 us, the dequant-reduce 259 against 270; 12 sources
// at 20 M elements 37.5 against 44.9 us, 4 sources at 100 M 102.7 against
// 109.5).
// WHOLE: the tile lies inside the array; otherwise (the last, partial tile)
// a group is clamped to the last one that starts inside and its second byte
// to the array's last, so that a partial tile keeps the batches in flight
// too; the values past the end are for the caller to drop.
template <int N, bool WHOLE, int G, class L>
__device__ __forceinline__ void i4grad_batch(f32x4 (&acc)[G], const L &from, uint32_t q0) {
    uint32_t w[N][G];
    float sc[N][G];
#pragma unroll
    for (int j = 0; j < N; ++j) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            w[j][g] = from.template codes<WHOLE>(q0 + j, g);
            sc[j][g] = from.scale(q0 + j, g);
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[g][e] = __builtin_fmaf(i4_code(w[j][g], e), sc[j][g], acc[g][e]);
}

// start of the group of four that holds element i, or of the last group
__device__ __forceinline__ uint32_t clamped_group(uint32_t i, uint32_t rest) {
    return i < rest ? i : (rest - 1) & ~3u;
}

// Where a lane's G groups of a tile find their codes and scales.
template <int G>
struct I4From {
    const I4Grad &s;
    size_t byte0;                // of the tile
    uint32_t byte[G], byte1[G];  // the groups' two bytes in it
    size_t k[G];                 // their blocks
    template <bool WHOLE>
    __device__ __forceinline__ uint32_t codes(uint32_t q, int g) const {
        const uint8_t *c = s.codes[q] + byte0;
        if constexpr (WHOLE)
            return ld_nt_at<uint16_t, 1>(c + byte[g]);
        else
            return c[byte[g]] | (uint32_t)c[byte1[g]] << 8;
    }
    __device__ __forceinline__ float scale(uint32_t q, int g) const { return s.scales[q][k[g]]; }
};

template <bool WHOLE, int G>
__device__ __forceinline__ I4From<G> i4_from(const I4Grad &s, size_t base, uint32_t lane,
                                             uint32_t rest) {
    I4From<G> f{s, base / 2};
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t i = g * 256 + lane * 4, c = WHOLE ? i : clamped_group(i, rest);
        f.byte[g] = c / 2;
        f.byte1[g] = WHOLE ? 0 : clamped(c / 2 + 1, (rest + 1) / 2);
        f.k[g] = block_of(s.block, base + c);
    }
    return f;
}

// The same P int4 copies interleaved in one receive buffer: for each block k
// of B elements the sources' codes lie side by side (source
// q's B/2 bytes at (k P + q) B/2) and so do their scales (source q's at
// k P + q).  P = 1 is the plain layout of one copy.  A wave's 256-element
// tile then reads all its codes within one run of P x 128 bytes (blocks of
// 256 or fewer) instead of from P separate arrays.  The gradient is formed in
// the same order with the same operations as from separate arrays, so the
// results are the same bits.
struct I4GradIl {
    const uint8_t *codes;
    const float *scales;
    uint32_t num_src;
    BlockDiv block;
    float scale_out;
};

// Byte offset of element i's code of source q, element i in block k (element
// i is in the low nibble when i is even).
__device__ __forceinline__ size_t il_code_byte(const I4GradIl &s, size_t i, size_t k,
                                               uint32_t q) {
    const size_t B = s.block.block;
    return (k * s.num_src + q) * (B / 2) + ((i - k * B) >> 1);
}

// The loads of the separate layout (a 2-byte code load and a scale per source),
// addressed in the interleaved buffer: a wave's loads of one source are 128
// contiguous bytes, and those of all sources lie within one run of the buffer.
// A group that starts inside the array lies inside the buffer whole (the
// buffer holds whole blocks), so a partial tile only clamps the group.
template <int G>
struct I4IlFrom {
    const uint8_t *base[G];  // the group's two bytes of source 0
    size_t stride;
    const float *scales[G];
    template <bool WHOLE>
    __device__ __forceinline__ uint32_t codes(uint32_t q, int g) const {
        return ld_nt_at<uint16_t, 1>(base[g] + q * stride);
    }
    __device__ __forceinline__ float scale(uint32_t q, int g) const { return scales[g][q]; }
};

template <bool WHOLE, int G>
__device__ __forceinline__ I4IlFrom<G> i4_from(const I4GradIl &s, size_t base, uint32_t lane,
                                               uint32_t rest) {
    I4IlFrom<G> f;
    f.stride = s.block.block / 2;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t i = g * 256 + lane * 4;
        const size_t e = base + (WHOLE ? i : clamped_group(i, rest));
        const size_t k = block_of(s.block, e);
        f.base[g] = s.codes + il_code_byte(s, e, k, 0);
        f.scales[g] = s.scales + k * s.num_src;
    }
    return f;
}

// The fp32 gradient array the separate partition step reads, behind the same
// interface.
struct F32Grad {
    const float *g;
};

// Many sources, a whole tile inside one block.  What bounds eight sources is
// HBM, what bounded many was latency: batch after batch of eight waited for
// its codes and scales, at the dozen waves per CU that suit the state's own
// streams.  So lane q holds source q's scale of the block (one load for up to
// 64 sources in place of one per source), each source's turn reads it from
// that lane into a scalar register, up to 32 sources' codes are in flight
// together, and short arrays leave residency to the hardware
// (receive_residency in zpp_chunk.h).  64 sources at 4,956,160 elements, receive
// step: separate arrays 73.9 -> 60.6 us, interleaved 66.9 -> 52.9 (43.6 at the
// copy rate); the dequant-reduce 80.5 -> 42.2 and 41.9 -> 38.2; 16 sources at
// 13 M: receive pass 101 -> 87 (separate), 87.5 -> 83.
// Codes of two groups by one 4-byte load, halves swapped between lane pairs,
// was no faster (62.8 and 59.1 us at 64 sources), nor was a cheaper decode
// (v_cvt_off_f32_i4 with the scale times 16).  The kernels hold 63 to 66
// registers in this form, but 82 to 128 with L2 decay from the interleaved buffer
// or two groups per lane (int8 blocks of 512), so 16 to 20 waves per CU where
// nothing caps them, which at 50 M elements and 16 sources is no slower than the
// form of few sources: the pass with L2 decay 318 us against 319.5, blocks of 512
// from separate arrays 343 against 348.
__device__ __forceinline__ float tile_scale(const I4Grad &s, size_t k, uint32_t lane) {
    return s.scales[lane < s.num_src ? lane : 0][k];
}
__device__ __forceinline__ float tile_scale(const I4GradIl &s, size_t k, uint32_t lane) {
    return s.scales[k * s.num_src + (lane < s.num_src ? lane : 0)];
}

struct TileCodes {
    const I4Grad &s;
    size_t byte;
    uint32_t lane;
    __device__ __forceinline__ uint32_t operator()(uint32_t q) const {
        return ld_nt_at<uint16_t, 1>(s.codes[q] + byte + 2 * lane);
    }
};
struct TileCodesIl {
    const uint8_t *base;
    uint32_t stride, lane;
    __device__ __forceinline__ uint32_t operator()(uint32_t q) const {
        return ld_nt_at<uint16_t, 1>(base + q * stride + 2 * lane);
    }
};
__device__ __forceinline__ TileCodes tile_codes(const I4Grad &s, size_t base, size_t,
                                                uint32_t lane) {
    return {s, base / 2, lane};
}
__device__ __forceinline__ TileCodesIl tile_codes(const I4GradIl &s, size_t base, size_t k,
                                                  uint32_t lane) {
    return {s.codes + il_code_byte(s, base, k, 0), s.block.block / 2, lane};
}

// N sources from q on, all loads in flight before the sums.  Not ALL: the
// first `count` of them; the loads past the last source repeat it.
template <int N, bool ALL, class F>
__device__ __forceinline__ void many_batch(f32x4 &acc, const F &codes, float scales, uint32_t q,
                                           uint32_t count) {
    uint32_t w[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
        w[j] = codes(ALL || j < (int)count ? q + j : q + count - 1);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (!ALL && j >= (int)count)
            break;
        const float sc = __uint_as_float(
            __builtin_amdgcn_readlane(__float_as_uint(scales), q + j));
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_fmaf(i4_code(w[j], e), sc, acc[e]);
    }
}

template <class GS>
__device__ __forceinline__ void many_sum(f32x4 &acc, const GS &s, size_t base, uint32_t lane) {
    const size_t k = block_of(s.block, base);
    const float scales = tile_scale(s, k, lane);
    const auto codes = tile_codes(s, base, k, lane);
    uint32_t q = 0;
    for (; q + 32 <= s.num_src; q += 32)
        many_batch<32, true>(acc, codes, scales, q, 32);
    if (q + 16 <= s.num_src) {
        many_batch<16, true>(acc, codes, scales, q, 16);
        q += 16;
    }
    if (q + 8 <= s.num_src) {
        many_batch<8, true>(acc, codes, scales, q, 8);
        q += 8;
    }
    if (q < s.num_src)
        many_batch<8, false>(acc, codes, scales, q, s.num_src - q);
}

// The gradients of a lane's G groups, r[g] of elements 256 g + 4 lane .. + 3
// of the tile of 256 G elements at `base`, `rest` of them inside the array
// (WHOLE: all).  MANY: the many-source form, where the tile allows it.
template <bool WHOLE, bool MANY, int G>
__device__ __forceinline__ void grad_tile(f32x4 (&r)[G], const F32Grad &s, size_t base,
                                          uint32_t lane, uint32_t rest) {
#pragma unroll
    for (int g = 0; g < G; ++g)
        r[g] = load4<WHOLE>(s.g + base, g * 256 + lane * 4, rest);
}

template <bool WHOLE, bool MANY, int G, class GS>
__device__ __forceinline__ void grad_tile(f32x4 (&r)[G], const GS &s, size_t base, uint32_t lane,
                                          uint32_t rest) {
#pragma unroll
    for (int g = 0; g < G; ++g)
        r[g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (MANY && WHOLE) {
#pragma unroll
        for (int g = 0; g < G; ++g)
            many_sum(r[g], s, base + g * 256, lane);
    } else {
        const auto from = i4_from<WHOLE, G>(s, base, lane, rest);
        uint32_t q0 = 0;
        for (; q0 + 8 <= s.num_src; q0 += 8)
            i4grad_batch<8, WHOLE>(r, from, q0);
        switch (s.num_src - q0) {
        case 1: i4grad_batch<1, WHOLE>(r, from, q0); break;
        case 2: i4grad_batch<2, WHOLE>(r, from, q0); break;
        case 3: i4grad_batch<3, WHOLE>(r, from, q0); break;
        case 4: i4grad_batch<4, WHOLE>(r, from, q0); break;
        case 5: i4grad_batch<5, WHOLE>(r, from, q0); break;
        case 6: i4grad_batch<6, WHOLE>(r, from, q0); break;
        case 7: i4grad_batch<7, WHOLE>(r, from, q0); break;
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            r[g][e] = i4grad_scaled(r[g][e], s.scale_out);
}

}  // namespace zpp
