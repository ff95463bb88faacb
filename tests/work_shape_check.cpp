// Host check of the work shapes for blocks that are not powers of two
// (zpp_chunk.h).
//
// Lane-group shapes (the int8 quantizer, 8 bf16 per vector, with and without
// the copy; the int4 quantizer, 4 fp32 per group), with the kernels' own
// parameters: the shape exists, G is 16, 32 or 64, S is at most 16 and at
// least the kernel's minimum where the fill allows it, the G S slots hold
// the block, and the walk -- block k in lanes [G (k % (64 /
// G)), +G) of a wave, lane r holding the block's vectors v G + r for v below
// the kernel's slot count (the power of two at or above S) -- covers every
// element exactly once, the last block cut short included.
//
// Workgroup renumbering per XCD (xcd_grouped): a permutation of [0, grid)
// for every grid and run length tried, and in every complete run of 8 R
// workgroups the ones that XCD x receives (positions x, x + 8, ...) take R
// consecutive numbers.
//
// Residency caps (residency_lds): for every count in use the reservation is
// whole LDS granules of the CU and holds exactly that many workgroups, with the
// wide kernel's own granule of LDS beside the rest too.
//
// Prints the worst fills and "work shapes ok".
#include <stdint.h>
#include <stdio.h>

#include <vector>

#include "zpp_chunk.h"

static uint32_t slot_bucket(uint32_t s, uint32_t smallest) {
    uint32_t b = smallest;
    while (b < s)
        b *= 2;
    return b;
}

static long check_groups(uint32_t w, uint32_t min_fill, uint32_t min_s, uint32_t smallest_bucket,
                         const char *what, double &worst) {
    long bad = 0;
    for (uint32_t b = 1; b <= 64; ++b) {
        if ((b & (b - 1)) == 0)
            continue;
        const uint32_t B = 64 * b, vpb = B / w;
        const zpp::GroupShape sh = zpp::group_shape(vpb, 16, min_fill, min_s);
        const bool pow2 = sh.G != 0 && (sh.G & (sh.G - 1)) == 0;
        if (!pow2 || sh.G < 16 || sh.G > 64 || sh.S == 0 || sh.S > 16 ||
            (uint64_t)sh.G * sh.S < vpb || (uint64_t)sh.G * (sh.S - 1) >= vpb) {
            printf("bad group shape: %s B %u -> G %u S %u\n", what, B, sh.G, sh.S);
            ++bad;
            continue;
        }
        const double fill = (double)vpb / ((double)sh.G * sh.S);
        if (fill < worst)
            worst = fill;
        // the rule: a shape with at least min_s slots and the fill asked for
        // is taken whenever one exists, the widest such group first
        for (uint32_t g = 64; g > sh.G; g /= 2) {
            const uint32_t s = (vpb + g - 1) / g;
            if (s >= min_s && s <= 16 && 100ull * vpb >= (uint64_t)min_fill * g * s) {
                printf("wider group passed over: %s B %u G %u (took %u)\n", what, B, g, sh.G);
                ++bad;
            }
        }
        const uint32_t slots = slot_bucket(sh.S, smallest_bucket);
        const uint32_t bpw = 64 / sh.G;
        // 2.5 waves of blocks, the last block short
        const uint64_t n = (uint64_t)B * (bpw * 2 + bpw / 2 + 1) - 3 * w - 1;
        std::vector<int> seen(n, 0);
        const uint64_t nblocks = (n + B - 1) / B;
        for (uint64_t k = 0; k < nblocks; ++k)
            for (uint32_t r = 0; r < sh.G; ++r)
                for (uint32_t v = 0; v < slots; ++v) {
                    const uint64_t j = (uint64_t)v * sh.G + r;
                    const uint64_t i = k * B + j * w;
                    if (j >= vpb || i >= n)
                        continue;
                    if (v >= sh.S) {
                        printf("slot past S holds data: %s B %u\n", what, B);
                        ++bad;
                    }
                    for (uint32_t e = 0; e < w && i + e < n; ++e)
                        ++seen[i + e];
                }
        for (uint64_t i = 0; i < n; ++i)
            if (seen[i] != 1) {
                printf("element %llu seen %d times: %s B %u\n", (unsigned long long)i, seen[i],
                       what, B);
                ++bad;
                break;
            }
    }
    return bad;
}

static long check_xcd_grouped() {
    long bad = 0;
    const size_t runs[] = {0, 1, 2, 4, 16, 128, 1000};
    const size_t grids[] = {1, 7, 8, 9, 63, 64, 65, 1023, 1024, 1025, 8 * 128 * 3 + 5, 99305};
    for (size_t R : runs)
        for (size_t grid : grids) {
            std::vector<int> seen(grid, 0);
            for (size_t w = 0; w < grid; ++w) {
                const size_t t = zpp::xcd_grouped(w, grid, R);
                if (t >= grid) {
                    printf("xcd_grouped out of range: R %zu grid %zu w %zu -> %zu\n", R, grid, w, t);
                    ++bad;
                    continue;
                }
                ++seen[t];
            }
            for (size_t t = 0; t < grid; ++t)
                if (seen[t] != 1) {
                    printf("xcd_grouped not a permutation: R %zu grid %zu\n", R, grid);
                    ++bad;
                    break;
                }
            if (R <= 1)
                continue;
            for (size_t run = 0; (run + 1) * 8 * R <= grid; ++run)
                for (size_t x = 0; x < 8; ++x)
                    for (size_t j = 0; j < R; ++j) {
                        const size_t w = run * 8 * R + x + 8 * j;
                        if (zpp::xcd_grouped(w, grid, R) != run * 8 * R + x * R + j) {
                            printf("xcd_grouped: XCD %zu not consecutive: R %zu grid %zu\n", x,
                                   R, grid);
                            ++bad;
                        }
                    }
        }
    return bad;
}

static long check_residency() {
    long bad = 0;
    for (int k : {2, 3, 4, 9, 10, 11, 12, 14, 16}) {
        const size_t lds = zpp::residency_lds(k);
        // 128 granules of 1280 bytes per CU
        const size_t held = 128 / ((lds + 1279) / 1280);
        if (lds % 1280 || lds > 64 * 1024 || held != (size_t)k ||
            zpp::workgroups_per_cu(lds) != held || zpp::workgroups_per_cu(lds - 1280 + 128) != held) {
            printf("residency: %zu bytes for %d hold %zu\n", lds, k, held);
            ++bad;
        }
    }
    if (zpp::residency_lds(0) != 0 || zpp::launch_lds(9, 32 * 256) != 0 ||
        zpp::launch_lds(9, 32 * 256 + 1) != zpp::residency_lds(9)) {
        printf("residency: launches left to the hardware\n");
        ++bad;
    }
    return bad;
}

// Runs per XCD of the refresh with its quantization: where they measure faster.
static long check_quant_copy_runs() {
    const struct {
        uint32_t block;
        size_t n;
        bool runs;
    } rule[] = {{64, 1, true},          {256, 4u << 20, true},   {512, 200u << 20, true},
                {1024, 4u << 20, false}, {4096, 50u << 20, false}, {192, 4u << 20, false},
                {576, 4u << 20, false},  {576, 32u << 20, true},  {960, (32u << 20) - 1, false},
                {1088, 200u << 20, false}, {4032, 50u << 20, false}};
    long bad = 0;
    // lane groups run per XCD in the instances of two slots alone
    for (uint32_t block = 192; block < 4096; block += 64)
        if ((block & (block - 1)) != 0 && zpp::quant_copy_runs(block, 200u << 20) &&
            zpp::group_shape(block / 8, 16, 55, 2).S > 2) {
            printf("runs of the copy: block %u has more than two slots\n", block);
            ++bad;
        }
    for (const auto &r : rule)
        if (zpp::quant_copy_runs(r.block, r.n) != r.runs) {
            printf("runs of the copy: block %u n %zu\n", r.block, r.n);
            ++bad;
        }
    return bad;
}

// Which fused steps give each block a workgroup of its own.
static long check_wide_block() {
    using zpp::Gradient;
    const size_t M = 1 << 20;
    const Gradient f32 = Gradient::kF32, sep = Gradient::kCopies, il = Gradient::kInterleaved;
    const struct {
        Gradient from;
        uint32_t num_src, block;
        size_t n;
        bool wide;
    } rule[] = {
        {f32, 0, 192, 8 * M, true},     {f32, 0, 192, 8 * M + 1, false},
        {f32, 0, 4096, M, true},        {f32, 0, 2048, 45 * M, false},
        {f32, 0, 832, 24 * M, true},    {f32, 0, 832, 32 * M, false},
        {f32, 0, 1280, 45 * M, false},  {f32, 0, 1024, 100 * M, true},
        {f32, 0, 1024, 128 * M, false}, {f32, 0, 1152, 100 * M, true},
        {sep, 8, 1024, 200 * M, true},  {il, 8, 1024, 200 * M, true},
        {il, 64, 1280, 20 * M, true},   {il, 32, 2048, 8 * M, true},
        {il, 16, 4096, 8 * M, false},   {sep, 64, 4096, 4 * M, true},
        {il, 15, 4096, 8 * M, true},    {il, 16, 192, M, true},
        {il, 16, 192, 6 * M, false},    {il, 31, 4032, 2 * M, true},
        {il, 32, 832, M, false},        {sep, 64, 832, M, true},
        {sep, 64, 4032, M, false},      {sep, 16, 832, 8 * M, true},
        {sep, 32, 832, 4 * M, false},   {sep, 16, 4032, 4 * M, false},
        {il, 64, 320, M, false},        {sep, 15, 832, 100 * M, true},
        {il, 8, 192, 2 * M, true},      {sep, 12, 192, 2 * M, true},
        {sep, 7, 192, 8 * M, true},     {sep, 8, 192, 6 * M, false},
        {sep, 15, 320, 8 * M, true},    {sep, 8, 320, 20 * M, false},
        {il, 3, 192, 8 * M, true},      {il, 4, 192, 6 * M, false},
        {il, 7, 320, 8 * M, true},      {il, 8, 448, 8 * M, false},
        {il, 15, 576, 8 * M, true},     {il, 8, 832, 16 * M, true},
        {il, 8, 832, 20 * M, false},    {il, 4, 1088, 52 * M, true},
        {il, 4, 1088, 100 * M, false},
    };
    long bad = 0;
    for (const auto &r : rule)
        if (zpp::wide_block(r.from, r.num_src, r.block, r.n) != r.wide) {
            printf("a workgroup per block: %d %u block %u n %zu\n", (int)r.from, r.num_src, r.block,
                   r.n);
            ++bad;
        }
    return bad;
}

// Residency with many int4 sources.
static long check_receive_residency() {
    using zpp::Gradient;
    const size_t M = 1 << 20;
    const struct {
        Gradient from;
        uint32_t num_src, grad_block;
        size_t n;
        bool quant;
        int want;
    } rule[] = {
        {Gradient::kInterleaved, 15, 256, 50 * M, true, 13},
        {Gradient::kInterleaved, 16, 256, 4 * M, true, 0},
        {Gradient::kInterleaved, 16, 256, 12 * M, true, 13},
        {Gradient::kInterleaved, 64, 1024, 20 * M, true, 13},
        {Gradient::kInterleaved, 24, 256, 50 * M, false, 11},
        {Gradient::kInterleaved, 16, 64, 4 * M, true, 0},
        {Gradient::kInterleaved, 16, 64, 8 * M, true, 13},
        {Gradient::kInterleaved, 32, 320, 8 * M, true, 0},
        {Gradient::kInterleaved, 32, 320, 50 * M, false, 13},
        {Gradient::kCopies, 15, 256, 50 * M, true, 13},
        {Gradient::kCopies, 16, 256, 12 * M - 1, true, 0},
        {Gradient::kCopies, 16, 256, 12 * M, true, 16},
        {Gradient::kCopies, 32, 64, 50 * M, true, 0},
        {Gradient::kCopies, 32, 1024, 50 * M, false, 16},
    };
    long bad = 0;
    for (const auto &r : rule)
        if (zpp::receive_residency(r.from, r.num_src, r.grad_block, r.n, r.quant, 13) != r.want) {
            printf("residency of a receive: %d %u %u %zu\n", (int)r.from, r.num_src, r.grad_block,
                   r.n);
            ++bad;
        }
    return bad;
}

// Residency of the step with its copies ahead of the quantizer.
static long check_copies_residency() {
    using zpp::Gradient;
    if (zpp::copies_residency(Gradient::kF32, 11) == 9 &&
        zpp::copies_residency(Gradient::kCopies, 12) == 12 &&
        zpp::copies_residency(Gradient::kInterleaved, 14) == 14)
        return 0;
    printf("residency of the copies\n");
    return 1;
}

// Tiles in flight of the int4 quantizer.
static long check_i4_tiles() {
    const size_t M = 1 << 20;
    const struct {
        uint32_t block, num_src;
        size_t n;
        bool two;
    } rule[] = {{256, 1, 8 * M, true},   {256, 8, 8 * M + 1, false}, {64, 1, 200 * M, false},
                {64, 2, 13 * M, false},  {64, 8, 20 * M, true},      {128, 2, 200 * M, false},
                {128, 4, 96 * M, false}, {128, 4, 128 * M, true},    {128, 8, 24 * M, false},
                {128, 8, 32 * M, true},  {128, 64, M, true}};
    long bad = 0;
    for (const auto &r : rule)
        if (zpp::i4_two_tiles(r.block, r.num_src, r.n) != r.two) {
            printf("int4 tiles: block %u senders %u n %zu\n", r.block, r.num_src, r.n);
            ++bad;
        }
    return bad;
}

// One-shot grids (for_tiles): the launches' tiles follow one another, cover the
// array with one partial tile at its very end, have workgroups enough for all of
// them and none to spare, and stay below 2^32 work-items each.  Sizes up to
// several launches (2^33 elements a launch for the step).
static long check_for_tiles() {
    const struct {
        uint32_t C, per_wg, threads;
    } shapes[] = {{256, 1, 64}, {512, 1, 64},  {512, 4, 256},  {2048, 1, 256}, {16384, 1, 256},
                  {320, 1, 128}, {4096, 1, 1024}, {1024, 4, 256}};
    long bad = 0;
    for (const auto &sh : shapes) {
        const size_t most = (((size_t)1 << 31) / sh.threads) * sh.per_wg * sh.C;
        for (size_t n : {(size_t)0, (size_t)1, (size_t)sh.C - 1, (size_t)sh.C, (size_t)sh.C + 1,
                         (size_t)sh.C * 7 + 5, most - 1, most, most + 1, most + sh.C,
                         2 * most - sh.C, 2 * most, 3 * most + 17}) {
            size_t next = 0, elems = 0, launches = 0;
            bool ok = true, ended = false;
            zpp::for_tiles(n, sh.C, sh.per_wg, sh.threads, true,
                           [&](const zpp::TileSpan &t, unsigned grid) {
                               const size_t count = (size_t)t.whole + (t.tail != 0);
                               ok = ok && !ended && t.first == next && count > 0 &&
                                    t.tail < sh.C && (size_t)grid * sh.threads < ((size_t)1 << 32) &&
                                    (size_t)grid * sh.per_wg >= count &&
                                    ((size_t)grid - 1) * sh.per_wg < count && t.on_lines == 1;
                               next += count;
                               elems += (size_t)t.whole * sh.C + t.tail;
                               ended = t.tail != 0;
                               ++launches;
                           });
            if (!ok || elems != n || launches != (n + most - 1) / most) {
                printf("tiles of %u: n %zu: %zu elements in %zu launches\n", sh.C, n, elems,
                       launches);
                ++bad;
            }
        }
    }
    return bad;
}

int main() {
    double worst_i8 = 1.0, worst_i8c = 1.0, worst_i4 = 1.0;
    long bad = 0;
    // the kernels' parameters: int8 fill 75% (55% with the copy), two slots
    // at least, slot instances 2 / 4 / 8 / 16; int4 fill 75%, three slots,
    // instances 4 / 8 / 16
    bad += check_groups(8, 75, 2, 2, "int8", worst_i8);
    bad += check_groups(8, 55, 2, 2, "int8+copy", worst_i8c);
    bad += check_groups(4, 75, 3, 4, "int4", worst_i4);
    bad += check_xcd_grouped();
    bad += check_for_tiles();
    bad += check_residency();
    bad += check_quant_copy_runs();
    bad += check_copies_residency();
    bad += check_wide_block();
    bad += check_i4_tiles();
    bad += check_receive_residency();
    printf("worst fill: int8 %.4f, int8+copy %.4f, int4 %.4f\n", worst_i8, worst_i8c, worst_i4);
    if (bad) {
        printf("%ld failures\n", bad);
        return 1;
    }
    printf("work shapes ok\n");
    return 0;
}
