// Work distribution shared by the kernels and the host checks: the lane
// layout of the quantizers for blocks that are not powers of two (any
// multiple of 64 up to 4096), the renumbering of workgroups per XCD, the tiles
// of a launch, the cap on workgroups resident per CU, and the rules by which a
// launch takes one form or another.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace zpp {

// Lane-group shape for blocks that are not powers of two: each block owns an
// aligned group of G lanes of a wave (G = 16, 32 or 64, so 64 / G blocks per
// wave), each lane holding S of the block's vectors (vector j of the block
// in lane j % G of the group, slot j / G); slots past the block's last
// vector stay empty.  The block's absmax is then a reduction over its G
// lanes with cross-lane xor shuffles, as in the power-of-two kernels.
// Chosen on the host: the largest G whose S (at least min_s, at most
// max_s) slots the block fills to at least min_fill_pct percent; failing
// that, the largest fill.  A block of more than 64 max_s vectors has no
// shape (G = 0).
struct GroupShape {
    uint32_t G;  // lanes per block
    uint32_t S;  // vector slots per lane
};

inline GroupShape group_shape(uint32_t vectors_per_block, uint32_t max_s, uint32_t min_fill_pct,
                              uint32_t min_s) {
    GroupShape best = {0, 0};
    uint64_t best_slots = 0;
    for (uint32_t g = 64; g >= 16; g /= 2) {
        const uint32_t s = (vectors_per_block + g - 1) / g;
        if (s > max_s)
            continue;
        if (s >= min_s && 100ull * vectors_per_block >= (uint64_t)min_fill_pct * g * s)
            return {g, s};
        // the same vectors in fewer slots is the larger fill
        if (best.G == 0 || (uint64_t)g * s < best_slots) {
            best = {g, s};
            best_slots = (uint64_t)g * s;
        }
    }
    return best;
}

// The dispatcher hands workgroups to the GPU's 8 XCDs in turn (workgroup w
// to XCD w % 8), each XCD with its own L2.  xcd_grouped(w, grid, R)
// renumbers workgroup w so that in every run of 8 R workgroups each XCD
// takes R consecutive positions (an incomplete last run keeps its order):
// neighbouring workgroups that read the same cache lines -- a line of
// per-block scales serving several tiles -- then fetch them through one L2.
// A permutation of [0, grid) for any R; R <= 1 is the identity.  (constexpr,
// so kernels and host checks call the same function.)
constexpr size_t xcd_grouped(size_t w, size_t grid, size_t R) {
    if (R <= 1)
        return w;
    const size_t run = w / (8 * R), r = w % (8 * R);
    return (run + 1) * 8 * R <= grid ? run * 8 * R + (r % 8) * R + r / 8 : w;
}

// The tiles of one launch: `whole` tiles of C elements from tile `first` on,
// then, where the array does not end with them, one of `tail` elements.  The
// host counts them, so that a kernel decides by one 32-bit comparison which
// kind its tile is.  (The remainder taken in the kernel as the smaller of two
// 64-bit values was compiled, in one kernel, to a select on a stale condition
// bit.)
struct TileSpan {
    size_t first;
    uint32_t whole;
    uint32_t tail;
    uint32_t on_lines;  // the outputs start on their lines (zpp_api.hip)
};

// One-shot grids over the tiles of C elements of an array of n, `per_wg` of
// them to a workgroup of `threads`, in as many launches as HIP's limit of
// 2^32 - 1 work-items per grid asks for: launch(tiles, workgroups).  A launch
// takes up to 2^31 work-items, so one-wave workgroups with a 256-element tile
// (the step) reach 2^33 elements before a second launch, the refresh 2^34.
// With no loop over tiles in the kernel the code of a whole tile is straight,
// and the rare partial tile's lies behind it.
template <class F>
void for_tiles(size_t n, uint32_t C, uint32_t per_wg, uint32_t threads, bool on_lines, F &&launch) {
    const size_t tiles = (n + C - 1) / C, most = (((size_t)1 << 31) / threads) * per_wg;
    for (size_t t = 0; t < tiles; t += most) {
        const size_t count = tiles - t < most ? tiles - t : most;
        const size_t whole = n / C - t < count ? n / C - t : count;
        launch(TileSpan{t, (uint32_t)whole, whole < count ? (uint32_t)(n % C) : 0u, on_lines},
               (unsigned)((count + per_wg - 1) / per_wg));
    }
}

// Whether the refresh with its quantization, its outputs off their lines, runs
// its workgroups per XCD.  With powers of two up to 512 it gains at every
// length (256 at 4 M, 8 elements into lines: 4.8 us, 5.1 in plain order; 131 M
// off by one 116, 123).  Larger blocks make tiles of 4096 elements and more,
// whose few shared lines don't pay for holding whole arrays apart by XCD (4096
// at 52 M: 56.5 us in runs, 52.3 plain).  Lane groups of other blocks gain over
// long arrays alone (576 at 4 M / 52 M / 210 M: 6.4 / 47.1 / 173 us in runs,
// 6.0 / 48.6 / 187 plain), and from 1024 on nothing (4032 at 52 M 55, 52.5).
inline bool quant_copy_runs(uint32_t block, size_t n) {
    if ((block & (block - 1)) == 0)
        return block <= 512;
    return block < 1024 && n >= ((size_t)32 << 20);
}

// Whether a wave of the int4 quantizer keeps two tiles in flight rather than
// four, for blocks up to 256.  Two put a short array on more waves (1 M: 3.3 us,
// 3.9 with four; 8 M 9.0, 13 M 12.9 and 12.4).  Blocks of 64 and 128 in a
// sender's slots, whose codes are runs of 32 and 64 bytes, take two over long
// arrays again (203 M, 8 senders: 64 286 -> 251 us, 128 187 -> 169), blocks of
// 128 the later the fewer senders share the buffer (two's time over four's: 64
// with 2 senders at 13 M 1.03, with 8 at 20 M .94; 128 with 8 senders at 13 M
// 1.03, 32 M .97; with 4 at 52 M 1.0; with 2 at 52 M 1.04, 90 M 1.04).
constexpr bool i4_two_tiles(uint32_t block, uint32_t num_src, size_t n) {
    if (n <= ((size_t)8 << 20))
        return true;
    if (block > 128 || num_src == 1)
        return false;
    if (block == 64)
        return n > ((size_t)13 << 20);
    return num_src > 2 && n > ((size_t)(num_src <= 4 ? 96 : 24) << 20);
}

// Residency cap.  The streaming kernels that keep many HBM streams open at
// once (the optimizer step: four arrays read, four written) run faster with
// fewer workgroups resident per CU than the hardware would otherwise place:
// too many waves in flight oversubscribe the memory channels.  A launch caps
// residency by reserving dynamic LDS that its kernel never touches, and the
// dispatcher still hands out the one-shot grid as workgroups retire.  A CU
// allocates LDS in granules (measured with a kernel that counts the
// workgroups alive at once: 128 granules of 1280 bytes), so residency_lds(k)
// is the fewest whole granules that k workgroups fit in and k + 1 do not.
// residency_lds(0) = 0 leaves residency to the hardware.
constexpr size_t kCUs = 256;          // CUs of an MI355X
constexpr size_t kLdsGranule = 1280;  // bytes
constexpr size_t kLdsGranules = 128;  // of one gfx950 CU: 160 KiB
constexpr size_t workgroups_per_cu(size_t lds) {
    return kLdsGranules / ((lds + kLdsGranule - 1) / kLdsGranule);
}
constexpr size_t residency_lds(int workgroups) {
    return workgroups <= 0 ? 0 : (kLdsGranules / (workgroups + 1) + 1) * kLdsGranule;
}
// The reservation of a launch of `wgs` one-wave workgroups.  A grid that fits
// the CUs' 32 wave slots at once has no workgroups left to hand out, so a cap
// only holds part of it back for a second round: it is left uncapped.  Capped
// -> uncapped at 1 M elements (4096 workgroups): Adam 6.5 -> 6.0 us, the fused
// step 7.7 -> 6.9, the receive step of 8 interleaved copies 7.6 -> 6.7; at 2 M
// (8192, the line) Adam 12.0 -> 12.1, fused 13.3 -> 13.5, the receive step
// 13.2 -> 12.6; at 4 M Adam 20.6 -> 21.4, the fused step 23.3 -> 24.4.
inline size_t launch_lds(int workgroups, size_t wgs) {
    return wgs <= 32 * kCUs ? 0 : residency_lds(workgroups);
}

// Where a step's gradient comes from: the fp32 array, the int4 copies as
// separate arrays, or those in one interleaved buffer.
enum class Gradient { kF32, kCopies, kInterleaved };

// The many-source form (zpp_i4grad.h): from this many sources on, with int4
// blocks that hold whole tiles.  With 12 it would gain at most 2% (receive step
// 78.5 against 78.9 us at 13 M elements) and the dequant-reduce would lose (57
// against 37.5 us at 20 M: its last, partial batch repeats loads); with 8 it
// loses everywhere (67.2 against 66.0).
constexpr uint32_t kManySources = 16;
constexpr bool many_sources(uint32_t num_src, uint32_t grad_block) {
    return num_src >= kManySources && grad_block % 256 == 0;
}

// Whether the fused step for a block other than 64, 128, 256 and 512 gives each
// block a workgroup of its own (fused_wide_kernel) rather than two kernels, the
// step with its copies and the quantizer.  What it costs is that a workgroup's
// waves start together and cover up to 16 neighbouring tiles on one XCD, which
// streams a few percent slower over long arrays than one-wave workgroups dealt
// out over the XCDs; what it saves is the second launch and 2 bytes read per
// element.  Measured against the two kernels, time over time:
//   fp32 gradient: every block gains up to 12 M elements (192 / 320 / 2048 /
//     4096 at 6 M .95 / .94 / .95 / .97, at 1 M .84 / .84 / .70 / .63) and
//     these lose at 45 M (1.04 / 1.02 / 1.02 / 1.06).  Blocks of 4 or 5 waves
//     gain for longer, by an amount that hangs on where the arrays lie and on
//     the card (arrays allocated one by one, three layouts on two cards): 1024 /
//     1088 / 1152 at 45 M .94 to 1.0 / .97 to 1.0 / .96 to .99, at 100 M .96 to
//     .98 / .99 to 1.03 / 1.0 to 1.05, at 128 M up to 1.07; the others at 25 M
//     832 1.0 to 1.03, 896 .98 to 1.01, 1280 .93 to .99, at 48 M up to 1.05 /
//     1.02 / 1.04.
//   int4 copies: a wave with idle lanes issues the loads of every source for
//     them too, and in such blocks the form has no many-source variant.  Up to
//     2 M elements it gains all the same below 32 sources (1 M, 16 interleaved
//     sources, 192 / 832 / 1344: 1.01 / .94 / .99; 12: 1.00 / .92 / .95), and in
//     blocks of 576 to 1344 from separate arrays with any number (32: .92 to
//     1.0).  Beyond, from 16 sources, it loses (4 M, 16 interleaved sources 192
//     / 832 / 1344: 1.13 / 1.01 / 1.01) but for those blocks from 16 to 31
//     separate arrays (8 M: .96 to 1.0).  Blocks of one or two waves, with no
//     neighbour to hide behind, lose sooner (8 M interleaved: 192 with 4 / 8
//     sources 1.04 / 1.09, 320 and 448 with 8 1.04; separate: 192 with 8 1.02,
//     320 .97).  Beyond 8 M, blocks of 832 to 1280: whole waves (1024 and 1280)
//     gain at every length (.93 to 1.0), the others from separate arrays below 16
//     sources too (.94 to 1.0), from the interleaved buffer with up to 4 sources
//     up to 64 M (.95 to 1.01) and otherwise up to 16 M (.95 to 1.0; 8 sources
//     at 52 M 1.03 to 1.05).  Blocks of 4096 and 16 sources lose from 8 M (1.0
//     to 1.05).
constexpr size_t kWideShort = (size_t)8 << 20;
constexpr bool wide_block(Gradient from, uint32_t num_src, uint32_t block, size_t n) {
    const bool four_waves = block > 768 && block <= 1280;
    if (from == Gradient::kF32) {
        if (!four_waves)
            return n <= kWideShort;
        return n <= (block >= 1024 && block <= 1152 ? 13 : 3) * kWideShort;
    }
    if (block % 256 == 0) {
        if (block > 2048 && num_src >= kManySources)
            return n <= kWideShort / 2;
        return four_waves || n <= kWideShort;
    }
    const bool medium = block > 512 && block <= 1344;
    if (n <= kWideShort / 4)
        return num_src < 2 * kManySources || (from == Gradient::kCopies && medium);
    if (num_src >= kManySources)
        return from == Gradient::kCopies && medium && num_src < 2 * kManySources &&
               n <= kWideShort;
    if (from == Gradient::kCopies)
        return four_waves || (n <= kWideShort && (block > 256 || num_src < 8));
    if (four_waves)
        return n <= (num_src <= 4 ? 8 : 2) * kWideShort;
    return n <= kWideShort && num_src < (block > 512 ? kManySources : block > 256 ? 8u : 4u);
}

// Workgroups per CU of the step with its copies alone, ahead of the quantizer
// over the primary it wrote; with_quant is the cap of the kernel that quantizes
// too.  The fp32 gradient keeps 9 (Llama-2-7B partition, both kernels: 1138 us
// with 9, 1146 with 10, 1154 with 11, 1153 with 8).  int4 copies keep as many as
// with the quantization: separate ones 291 us with 12, 299 with 9; interleaved
// ones, 14 against 9, 1 copy at 50 M 273 / 280, 4 at 20 M 117 / 120, 9 to 15 from
// 33 M on 1.0 / 1.1 times (12 at 100 M 633 / 706).  Eight at 100 M went either way
// by the card (572 / 597, 606 / 596).
constexpr int copies_residency(Gradient from, int with_quant) {
    return from == Gradient::kF32 ? 9 : with_quant;
}

// Workgroups per CU of a step that receives num_src int4 copies; few is the
// kernel's cap for few of them.  With many sources a short array waits on the
// latency of their loads and takes every wave the hardware holds (64
// interleaved sources at 4.7 M, receive step: 51.3 us uncapped, 53.1 capped); a
// long one streams, and from the interleaved buffer keeps the cap (uncapped /
// capped, 16 sources at 50 M: blocks of 256 302.6 / 285, of 64 349 / 332, of
// 320 359 / 343; 64 sources at 8 M, blocks of 64 and 320: capped better and
// worse by 3%).  Separate arrays in the many-source form stream best with 16 (16
// sources, blocks of 1024 at 50 M: 319 uncapped, 308, 325 with the cap of few
// sources); in other blocks every cap loses (32 sources, blocks of 64 at 50 M
// 391 / 435).  The step with its copies alone
// (quant false) keeps 11 in the many-source form of the interleaved buffer (24
// sources at 50 M, both kernels: 385 uncapped, 393 with 9, 365).
constexpr int receive_residency(Gradient from, uint32_t num_src, uint32_t grad_block, size_t n,
                                bool quant, int few) {
    if (num_src < kManySources)
        return few;
    const bool many = many_sources(num_src, grad_block);
    if (from == Gradient::kCopies)
        return many && n >= ((size_t)12 << 20) ? 16 : 0;
    if (n < ((size_t)(grad_block < 256 ? 8 : 12) << 20))
        return 0;
    return many && !quant ? 11 : few;
}

}  // namespace zpp
