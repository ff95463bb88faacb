// Host check of the workgroup order that the C ABI asks of each launch: runs
// per XCD where an output starts off its line, plain order otherwise.  The
// library's zpp_api.hip is linked with stand-ins for the kernel launchers that
// record the flag; the addresses are only compared, so no device is needed.
//
// Every call is made with all arrays the same number of elements into lines of
// 128 bytes, the way one layer's range of flat buffers lies, and with one
// array at a time moved.  Prints "launch order ok".
#include <stdint.h>
#include <stdio.h>

#include "zpp.h"
#include "zpp_launch.h"

namespace {
int lines = -1;
hipError_t record(bool on_lines) {
    lines = on_lines;
    return hipSuccess;
}
}  // namespace

namespace zpp {
hipError_t launch_adam(float *, float *, float *, const float *, uint16_t *, size_t,
                       const AdamConsts &, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_refresh(uint16_t *, const uint16_t *, size_t, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_quantize(const uint16_t *, size_t, uint32_t, int8_t *, float *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_quantize_copy(const uint16_t *, size_t, uint32_t, int8_t *, float *, uint16_t *,
                                bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_fused(float *, float *, float *, const float *, uint16_t *, uint16_t *, int8_t *,
                        float *, size_t, uint32_t, const AdamConsts &, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_gather(const GatherShards &, uint32_t, size_t, uint32_t, size_t, uint16_t *,
                         bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_quantize_i4(const float *, size_t, uint32_t, uint8_t *, float *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_dequant_reduce_i4(const uint8_t *const *, const float *const *, uint32_t, size_t,
                                    uint32_t, float, float *, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_fused_receive(float *, float *, float *, const uint8_t *const *,
                                const float *const *, uint32_t, uint32_t, float, uint16_t *,
                                uint16_t *, int8_t *, float *, size_t, uint32_t,
                                const AdamConsts &, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_receive_adam(float *, float *, float *, const uint8_t *const *,
                               const float *const *, uint32_t, uint32_t, float, uint16_t *, size_t,
                               const AdamConsts &, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_quantize_i4_il(const float *, size_t, uint32_t, uint32_t, uint32_t, uint8_t *,
                                 float *, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_dequant_reduce_i4_il(const uint8_t *, const float *, uint32_t, size_t, uint32_t,
                                       float, float *, bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_receive_adam_il(float *, float *, float *, const uint8_t *, const float *,
                                  uint32_t, uint32_t, float, uint16_t *, size_t, const AdamConsts &,
                                  bool l, hipStream_t) {
    return record(l);
}
hipError_t launch_fused_receive_il(float *, float *, float *, const uint8_t *, const float *,
                                   uint32_t, uint32_t, float, uint16_t *, uint16_t *, int8_t *,
                                   float *, size_t, uint32_t, const AdamConsts &, bool l,
                                   hipStream_t) {
    return record(l);
}
}  // namespace zpp

namespace {

size_t N;
enum { kMaster, kM, kV, kPrimary, kSecondary, kCodes, kOut, kArrays };
const size_t kBytes[kArrays] = {4, 4, 4, 2, 2, 1, 4};  // of an element
size_t at[kArrays];                                    // elements into a line

void *region(unsigned k) { return (void *)(uintptr_t)((16ull << 30) + ((uint64_t)k << 30)); }
char *array(int a) { return (char *)region(a) + at[a] * kBytes[a]; }

long bad = 0;

void expect(const char *call, zpp_status st, bool want) {
    if (st != ZPP_OK || lines != (int)want) {
        printf("%s: status %d, order flag %d, expected %d; elements into lines:", call, (int)st,
               lines, (int)want);
        for (size_t x : at)
            printf(" %zu", x);
        printf("\n");
        ++bad;
    }
    lines = -1;
}

bool on(int a, size_t line) { return at[a] * kBytes[a] % line == 0; }

void check() {
    const zpp_adam_hparams hp = {1e-4f, 0.9f, 0.95f, 1e-8f, 0.1f, 1, 1};
    float *p = (float *)array(kMaster), *m = (float *)array(kM), *v = (float *)array(kV);
    uint16_t *pr = (uint16_t *)array(kPrimary), *se = (uint16_t *)array(kSecondary);
    int8_t *c = (int8_t *)array(kCodes);
    float *out = (float *)array(kOut), *g = (float *)region(20), *sc = (float *)region(21);
    const uint8_t *x = (const uint8_t *)region(22);
    const float *xs = (const float *)region(23);
    const uint8_t *xl[1] = {x};
    const float *xsl[1] = {xs};

    const bool step = on(kMaster, 128) && on(kM, 128) && on(kV, 128);
    expect("adam", zpp_adam_partition_step(p, m, v, g, pr, N, &hp, nullptr),
           step && on(kPrimary, 64));
    expect("receive", zpp_qgz_receive_adam_step(p, m, v, xl, xsl, 1, 256, 1.0f, pr, N, &hp,
                                                nullptr, nullptr, 0, nullptr),
           step && on(kPrimary, 64));
    expect("receive interleaved",
           zpp_qgz_receive_adam_step_interleaved(p, m, v, x, xs, 1, 256, 1.0f, pr, N, &hp, nullptr,
                                                 nullptr, 0, nullptr),
           step && on(kPrimary, N <= (2u << 20) ? 128 : 64));
    const bool all = step && on(kPrimary, 128) && on(kSecondary, 128) && on(kCodes, 64);
    expect("fused",
           zpp_adam_step_refresh_quantize(p, m, v, g, pr, se, c, sc, N, 256, &hp, nullptr, nullptr,
                                          nullptr),
           all);
    expect("fused without a secondary",
           zpp_adam_step_refresh_quantize(p, m, v, g, pr, nullptr, c, sc, N, 256, &hp, nullptr,
                                          nullptr, nullptr),
           step && on(kPrimary, 128) && on(kCodes, 64));
    expect("pass",
           zpp_qgz_receive_step_refresh_quantize(p, m, v, xl, xsl, 1, 256, 1.0f, pr, se, c, sc, N,
                                                 256, &hp, nullptr, nullptr, 0, nullptr),
           all);
    expect("pass interleaved",
           zpp_qgz_receive_step_refresh_quantize_interleaved(p, m, v, x, xs, 1, 256, 1.0f, pr, se,
                                                             c, sc, N, 256, &hp, nullptr, nullptr,
                                                             0, nullptr),
           all);
    expect("refresh", zpp_refresh_secondary(se, (const uint16_t *)g, N, nullptr, nullptr, nullptr),
           on(kSecondary, 128));
    expect("refresh and quantize",
           zpp_refresh_quantize_i8(se, (const uint16_t *)g, N, 256, c, sc, nullptr, nullptr,
                                   nullptr),
           on(kSecondary, 128) && on(kCodes, 64));
    expect("refresh and quantize in blocks of 192",
           zpp_refresh_quantize_i8(se, (const uint16_t *)g, N, 192, c, sc, nullptr, nullptr,
                                   nullptr),
           on(kSecondary, 128) && on(kCodes, 128));
    expect("reduce",
           zpp_dequant_reduce_i4(xl, xsl, 1, N, 256, 1.0f, out, nullptr, nullptr, 0, nullptr),
           on(kOut, 32));
    expect("reduce interleaved",
           zpp_dequant_reduce_i4_interleaved(x, xs, 1, N, 256, 1.0f, out, nullptr, nullptr, 0,
                                             nullptr),
           on(kOut, 32));
    const int8_t *sl[2] = {(const int8_t *)x, (const int8_t *)x};
    const float *ssl[2] = {xs, xs};
    for (size_t shard : {N, N + 8})
        expect("gather",
               zpp_dequant_gather_layer(sl, ssl, 2, shard, 256, 2 * shard, pr, nullptr, nullptr, 0,
                                        nullptr),
               on(kPrimary, 32) && shard % 16 == 0);
}

void check_order() {
    for (size_t elems : {0, 1, 4, 8, 16, 32, 64, 128, 129}) {
        for (size_t &x : at)
            x = elems;
        check();
        for (size_t &x : at) {  // one array moved
            x = 0;
            check();
            x = elems;
        }
    }
    for (size_t elems : {1, 4, 8, 16, 32, 64}) {  // one array off
        for (size_t &x : at)
            x = 0;
        for (size_t &x : at) {
            x = elems;
            check();
            x = 0;
        }
    }
}

}  // namespace

int main() {
    for (size_t n : {4096, 2 << 20, (2 << 20) + 256}) {
        N = n;
        check_order();
    }
    if (bad) {
        printf("%ld failures\n", bad);
        return 1;
    }
    printf("launch order ok\n");
    return 0;
}
