// Device-side helpers shared by the partition-path kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "zpp_chunk.h"
#include "zpp_launch.h"

namespace zpp {

constexpr int kWave = 64;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// float -> bf16 bits, round to nearest even.  Adding 0x7FFF plus the lowest
// kept bit carries into the kept half exactly when the dropped half is above
// one half ulp, or exactly one half with an odd kept half.  NaN maps to the
// canonical 0x7FC0; +-Inf and overflow come out as +-Inf by the same carry.
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? 0x7FC0u : r;
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return bf16_rne_bits(lo) | (bf16_rne_bits(hi) << 16);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Block index of element i (BlockDiv, zpp_launch.h): the branch is uniform
// across a launch.
__device__ __forceinline__ size_t block_of(const BlockDiv &d, size_t i) {
    return d.magic ? (size_t)__umul64hi((unsigned long long)(i >> 6), d.magic) : i >> d.shift;
}

// Ranges that do not start on a 128-byte line: a tile's accesses end inside
// lines that the next tile goes on with, and where two XCDs take the two, each
// fetches the shared lines from memory.  So neighbouring tiles run on one XCD, in
// runs of this many, and meet in its L2.  Counters at 13.1 M elements off by one,
// read and written, plain order / runs (algorithmic): Adam 236 / 210 (210) and 190
// / 191 (184) MB, the fused step 236 / 211 and 234 / 235 (223), a bf16 copy 29.5 /
// 26.3 (26.2) and 27 / 27.  The Adam step there 81.3 us without, 70.2 / 69.6 /
// 69.3 / 68.9 with runs of 16 / 32 / 64 / 128 (100 M: 618, 543 / 531 / 518 /
// 511), the fused step 105 and 80, the receive step 82 and 72, the gather of
// 200 M 121 and 102.  (Outputs that start inside a line but far enough from its
// ends lose by the runs: zpp_api.hip has the measured lines.)  Stored as ordinary,
// temporal ones they were slower (73 us for the Adam step, 95 without the runs).
constexpr size_t kOffLineXcdRun = 128;

// The tile of workgroup w of the launch: renumbered in runs of `run` per XCD
// where the outputs start on lines.
__device__ __forceinline__ uint32_t tile_of(uint32_t w, uint32_t grid, const TileSpan &tiles,
                                            size_t run) {
    return (uint32_t)(tiles.on_lines ? xcd_grouped(w, grid, run)
                                     : xcd_grouped(w, grid, kOffLineXcdRun));
}

// Streaming accesses: every byte is touched once, so loads and stores are
// marked non-temporal.
template <typename T>
__device__ __forceinline__ T ld_nt(const T *p) {
    return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void st_nt(T *p, T v) {
    __builtin_nontemporal_store(v, p);
}

// The same for vectors at addresses that are aligned to an element (A bytes)
// and no further: the hardware takes vector accesses of global memory at any
// address, so one kernel serves every alignment.  Kernels of their own for
// arrays off the vectors' alignment, an element at a time, took at 13.1 M
// elements off by one (us, against these accesses): the int8 quantizer 23.3
// (10.0), the dequant-reduce of 8 copies 110 (30), the receive step 165 (72),
// the fused step 126 (80), the gather of 16.8 M 29.1 (10.8).
template <class V, int A>
__device__ __forceinline__ V ld_nt_at(const void *p) {
    typedef V U __attribute__((aligned(A)));
    return __builtin_nontemporal_load(reinterpret_cast<const U *>(p));
}
template <class V, int A>
__device__ __forceinline__ void st_nt_at(void *p, V v) {
    typedef V U __attribute__((aligned(A)));
    __builtin_nontemporal_store(v, reinterpret_cast<U *>(p));
}

// Four consecutive elements i .. i+3 of a tile whose arrays start at p and
// hold r >= 1 elements (p is the same for the whole wave, so the offset stays
// 32 bits beside a scalar base).  WHOLE: the tile lies inside the arrays, one
// vector access.  Otherwise (a launch's last, partial tile) every element is
// its own load at an index clamped into the array, and only the elements
// inside are stored.  The four loads depend on nothing, so the lanes of a
// partial tile pay one memory latency for all their arrays rather than one
// per element: with the elements taken one after the other, the last tile
// alone outlasted a short launch (the single receive pass of 64 sources at
// 4,956,320 elements: 115.8 us, 88.2 us at 4,956,160, which is whole tiles).
__device__ __forceinline__ uint32_t clamped(uint32_t i, uint32_t r) { return i < r ? i : r - 1; }

template <bool WHOLE>
__device__ __forceinline__ f32x4 load4(const float *p, uint32_t i, uint32_t r) {
    if constexpr (WHOLE)
        return ld_nt_at<f32x4, 4>(p + i);
    else
        return f32x4{p[clamped(i, r)], p[clamped(i + 1, r)], p[clamped(i + 2, r)],
                     p[clamped(i + 3, r)]};
}

template <bool WHOLE>
__device__ __forceinline__ void store4(float *p, uint32_t i, uint32_t r, const f32x4 &v) {
    if constexpr (WHOLE) {
        st_nt_at<f32x4, 4>(p + i, v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < r)
                p[i + e] = v[e];
    }
}

// four bf16 packed in two words
template <bool WHOLE>
__device__ __forceinline__ void store4_bf16(uint16_t *p, uint32_t i, uint32_t r, const u32x2 &v) {
    if constexpr (WHOLE) {
        st_nt_at<u32x2, 2>(p + i, v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < r)
                p[i + e] = (uint16_t)(v[e / 2] >> (16 * (e % 2)));
    }
}

// four int8 packed in a word
template <bool WHOLE>
__device__ __forceinline__ void store4_i8(int8_t *p, uint32_t i, uint32_t r, uint32_t v) {
    if constexpr (WHOLE) {
        st_nt_at<uint32_t, 1>(p + i, v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < r)
                p[i + e] = (int8_t)((v >> (8 * e)) & 0xFFu);
    }
}

}  // namespace zpp
