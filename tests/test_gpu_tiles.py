"""GPU checks of the kernels' tile edges and dispatch rules: every result of a
call equals, bit for bit, the one the same elements get from a call that takes
another route (whole tiles, other alignment), and nothing past the end of an
output is written.  The routes compared against are themselves checked against
the oracle by the other GPU tests."""
import numpy as np
import pytest
import torch

from paper_2407_01614_amd import synth

pytestmark = pytest.mark.gpu

HP = dict(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-6, weight_decay=0.5)
GUARD = 64


@pytest.fixture(scope="module")
def zpp():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_01614_amd import zpp as mod
    return mod


class Buf:
    """`n` elements, `offset` elements into a buffer that goes on for GUARD
    bytes behind them, filled with 0x5A."""

    def __init__(self, n, dtype, offset=0, values=None):
        self.size = torch.empty(0, dtype=dtype).element_size()
        self.raw = torch.full(((n + offset) * self.size + GUARD,), 0x5A, dtype=torch.uint8,
                              device="cuda")
        self.end = (n + offset) * self.size
        self.lo = offset * self.size
        self.t = self.raw[:self.end].view(dtype)[offset:]
        if values is not None:
            self.t.copy_(torch.from_numpy(values)[:n])

    def bits(self):
        assert (self.raw[:self.lo] == 0x5A).all() and (self.raw[self.end:] == 0x5A).all(), \
            "written outside the array"
        return self.raw[self.lo:self.end].cpu().numpy()


def state(n, full, offset=0):
    p = synth.master_weights(full, 300)
    m, v = synth.moments(full, 300)
    return [Buf(n, torch.float32, offset, a) for a in (p, m, v)] + [Buf(n, torch.int16, offset)]


def copies(zpp, full, k, block, interleaved):
    """k int4 copies of `full` elements, as the interleaved buffer or as lists."""
    x = [torch.from_numpy(synth.gradients(full, 301, q)).cuda() for q in range(k)]
    if interleaved:
        nc, ns = zpp.interleaved_sizes(full, block, k)
        codes = torch.zeros(nc, dtype=torch.uint8, device="cuda")
        scales = torch.zeros(ns, device="cuda")
        for q in range(k):
            zpp.quantize_blockwise_i4_interleaved(x[q], codes, scales, source=q, num_src=k,
                                                  block=block)
        return codes, scales
    codes = [torch.zeros((full + 1) // 2, dtype=torch.uint8, device="cuda") for _ in range(k)]
    scales = [torch.zeros(-(-full // block), device="cuda") for _ in range(k)]
    for q in range(k):
        zpp.quantize_blockwise_i4(x[q], codes[q], scales[q], block=block)
    return codes, scales


def receive(zpp, n, full, src, k, block, interleaved, single_pass, offset=0):
    """The receive step of n elements from copies of `full`, into guarded
    buffers: their bits, the int8 codes and scales last for the single pass."""
    st = state(n, full, offset)
    codes, scales = src
    if not interleaved:  # exactly the bytes that n elements have
        codes = [Buf((n + 1) // 2, torch.uint8, 0, c[:(n + 1) // 2].cpu().numpy()).t
                 for c in codes]
    args = [b.t for b in st[:3]] + [codes, scales] + ([k] if interleaved else []) + [st[3].t]
    kw = dict(HP, step=3, scale_out=1.0 / k, n=n)
    if not single_pass:
        call = (zpp.qgz_receive_adam_step_interleaved if interleaved
                else zpp.qgz_receive_adam_step)
        call(*args, block=block, **kw)
        return [b.bits() for b in st]
    out = [Buf(n, torch.int16, offset), Buf(n, torch.int8, offset),
           Buf(-(-n // 256), torch.float32)]
    call = (zpp.qgz_receive_step_refresh_quantize_interleaved if interleaved
            else zpp.qgz_receive_step_refresh_quantize)
    call(*args, *[b.t for b in out], grad_block=block, block=256, **kw)
    return [b.bits() for b in st + out]


def same_start(got, ref, n, names):
    for g, r, name in zip(got, ref, names):
        assert np.array_equal(g, r[:g.size]), "%s at n = %d" % (name, n)


NAMES = ("master", "exp_avg", "exp_avg_sq", "primary", "secondary")


@pytest.mark.parametrize("interleaved", [False, True], ids=["separate", "interleaved"])
@pytest.mark.parametrize("k,block", [(1, 64), (3, 256), (8, 192), (19, 256), (64, 512)])
def test_partial_tiles(zpp, k, block, interleaved):
    """A last tile that is not whole: each element as in a call of whole
    tiles, and the int8 quantization of the short block as the quantizer
    gives it for the primary that the pass wrote."""
    full = 1024
    src = copies(zpp, full, k, block, interleaved)
    whole = receive(zpp, full, full, src, k, block, interleaved, False)
    reduce = zpp.dequant_reduce_i4_interleaved if interleaved else zpp.dequant_reduce_i4
    sum_args = (src[0], src[1]) + ((k,) if interleaved else ())
    g = Buf(full, torch.float32)
    reduce(*sum_args, full, g.t, block=block, scale_out=1.0 / k)
    for n in (1, 2, 3, 5, 255, 257, 258, 259, 511, 512, 514, 767, 1021):
        same_start(receive(zpp, n, full, src, k, block, interleaved, False), whole, n, NAMES)
        got = receive(zpp, n, full, src, k, block, interleaved, True)
        same_start(got[:4] + [got[4]], whole + [whole[3]], n, NAMES)
        primary = torch.from_numpy(got[3].view(np.int16)).cuda()
        codes, scales = Buf(n, torch.int8), Buf(-(-n // 256), torch.float32)
        zpp.quantize_blockwise_i8(primary, codes.t, scales.t, block=256)
        assert np.array_equal(got[5], codes.bits()) and np.array_equal(got[6], scales.bits()), n
        s = Buf(n, torch.float32)
        reduce(*sum_args, n, s.t, block=block, scale_out=1.0 / k)
        same_start([s.bits()], [g.bits()], n, ("reduced",))
        # the step from that gradient, and the pass with it
        st = state(n, full)
        zpp.adam_partition_step(*[b.t for b in st[:3]], s.t, st[3].t, step=3, **HP)
        same_start([b.bits() for b in st], whole, n, NAMES)


@pytest.mark.parametrize("interleaved", [False, True], ids=["separate", "interleaved"])
@pytest.mark.parametrize("k,n,block", [(15, 1029, 256), (16, 1029, 256), (23, 1029, 512),
                                       (31, 1029, 256), (33, 1029, 768), (45, 1029, 192),
                                       (63, 1029, 256), (16, 4194304 + 258, 256),
                                       (5, 2053, 256), (6, 2053, 320), (7, 2053, 256)])
def test_source_counts(zpp, k, n, block, interleaved):
    """Every batch length of the int4 sources, below and from the count that
    takes the many-source form, against the oracle bit for bit; scales that
    are zero, subnormal, huge, infinite and NaN among them."""
    import oracle
    codes = [synth.rng(302, 0, q).integers(0, 256, (n + 1) // 2, dtype=np.uint8)
             for q in range(k)]
    nb = -(-n // block)
    scales = [synth.random_scales(nb, 303, q) for q in range(k)]
    for q, bad in enumerate((0.0, 1e-45, 3e38, np.inf, np.nan)):
        scales[q % k][min(q, nb - 1)] = bad
    ref = oracle.dequant_reduce_i4(codes, scales, n, block, 1.0 / 3.0)
    out = Buf(n, torch.float32)
    if interleaved:
        c = np.zeros((nb, k, block // 2), np.uint8)
        for q in range(k):
            flat = np.zeros(nb * block // 2, np.uint8)
            flat[:codes[q].size] = codes[q]
            c[:, q] = flat.reshape(nb, -1)
        zpp.dequant_reduce_i4_interleaved(
            torch.from_numpy(c.reshape(-1)).cuda(),
            torch.from_numpy(np.stack(scales, 1).reshape(-1)).cuda(), k, n, out.t, block=block,
            scale_out=float(np.float32(1.0 / 3.0)))
    else:
        zpp.dequant_reduce_i4([torch.from_numpy(c).cuda() for c in codes],
                              [torch.from_numpy(s).cuda() for s in scales], n, out.t, block=block,
                              scale_out=float(np.float32(1.0 / 3.0)))
    got = out.bits().view(np.float32)
    nan = np.isnan(ref)
    assert nan.any() and np.array_equal(nan, np.isnan(got))
    assert np.array_equal(got[~nan].view(np.uint32), ref[~nan].view(np.uint32))


def every_call(zpp, n, block, offset, interleaved):
    """Each call once with every array `offset` elements into its buffer: the
    bits of all its outputs."""
    got = {}

    def arrays(*specs):
        return [Buf(m, dt, offset, v) for m, dt, v in specs]

    def take(name, bufs):
        got.update({"%s[%d]" % (name, i): b.bits() for i, b in enumerate(bufs)})

    nb = -(-n // block)
    f32, i16, i8, u8 = torch.float32, torch.int16, torch.int8, torch.uint8
    g, w = synth.gradients(n, 310), synth.bf16_weights(n, 311).view(np.int16)
    st = state(n, n, offset)
    gb, = arrays((n, f32, g))
    zpp.adam_partition_step(*[b.t for b in st[:3]], gb.t, st[3].t, step=3, **HP)
    take("adam", st)
    st, out = state(n, n, offset), arrays((n, i16, None), (n, i8, None), (nb, f32, None))
    zpp.adam_step_refresh_quantize(*[b.t for b in st[:3]], gb.t, st[3].t, *[b.t for b in out],
                                   block=block, step=3, **HP)
    take("fused", st + out)
    wb, = arrays((n, i16, w))
    out = arrays((n, i16, None), (n, i8, None), (nb, f32, None))
    zpp.refresh_quantize_i8(out[0].t, wb.t, out[1].t, out[2].t, block=block)
    take("refresh_quantize", out)
    out = arrays((n, i16, None))
    zpp.refresh_secondary(out[0].t, wb.t)
    take("refresh", out)
    out = arrays((n, i8, None), (nb, f32, None))
    zpp.quantize_blockwise_i8(wb.t, out[0].t, out[1].t, block=block)
    take("quantize_i8", out)
    layer = arrays((2 * n - 3, i16, None))
    zpp.dequant_gather_layer([out[0].t, out[0].t], [out[1].t, out[1].t], n, 2 * n - 3, layer[0].t,
                             block=block)
    take("gather", layer)
    k = 3
    if interleaved:
        nc, ns = zpp.interleaved_sizes(n, block, k)
        codes, scales = arrays((nc, u8, np.zeros(nc, np.uint8)), (ns, f32, np.zeros(ns, np.float32)))
        for q in range(k):
            zpp.quantize_blockwise_i4_interleaved(gb.t, codes.t, scales.t, source=q, num_src=k,
                                                  block=block)
        take("quantize_i4", (codes, scales))
        src, reduce, step = ((codes.t, scales.t, k), zpp.dequant_reduce_i4_interleaved,
                             zpp.qgz_receive_adam_step_interleaved)
    else:
        copies = [arrays(((n + 1) // 2, u8, None), (nb, f32, None)) for _ in range(k)]
        for c, s in copies:
            zpp.quantize_blockwise_i4(gb.t, c.t, s.t, block=block)
            take("quantize_i4", (c, s))
        src, reduce, step = (([c.t for c, _ in copies], [s.t for _, s in copies]),
                             zpp.dequant_reduce_i4, zpp.qgz_receive_adam_step)
    out = arrays((n, f32, None))
    reduce(*src, n, out[0].t, block=block, scale_out=0.5)
    take("reduce", out)
    st = state(n, n, offset)
    step(*[b.t for b in st[:3]], *src, st[3].t, block=block, scale_out=0.5, step=3, **HP)
    take("receive", st)
    return got


@pytest.mark.parametrize("interleaved", [False, True], ids=["separate", "interleaved"])
@pytest.mark.parametrize("n,block", [(2051, 256), (300 * 256 + 7, 64), (263001, 320), (9999, 4096)])
def test_alignments(zpp, n, block, interleaved):
    """Arrays that start off a vector's alignment, on it but off a cache line,
    and on a line: the same bits, and nothing outside the arrays written.
    (263,001 elements are more tiles than one run of workgroups per XCD.)"""
    ref = every_call(zpp, n, block, 0, interleaved)
    for offset in (1, 2, 3, 5, 8, 32, 64, 128):
        got = every_call(zpp, n, block, offset, interleaved)
        for name, r in ref.items():
            assert np.array_equal(got[name], r), (name, offset)


@pytest.mark.parametrize("block", [192, 320, 576, 960, 1088])
def test_refresh_quantize_long_ranges_off_lines(zpp, block):
    """The refresh with its quantization over ranges off their lines, around
    the length from which lane groups run per XCD (a run is 1024 workgroups of
    4 to 16 blocks): what the call gives for arrays on lines."""
    limit = 32 << 20
    gen = torch.Generator(device="cuda").manual_seed(block)
    src = torch.empty(limit + 2051, device="cuda").normal_(0, 0.02, generator=gen).bfloat16()
    for n in (limit - 1, limit, limit + 2051):
        nb = -(-n // block)
        got = []
        for offset in (0, 3, 8):
            x = Buf(n, torch.bfloat16, offset)
            x.t.copy_(src[:n])
            out = [Buf(n, torch.bfloat16, offset), Buf(n, torch.int8, offset),
                   Buf(nb, torch.float32)]
            zpp.refresh_quantize_i8(out[0].t, x.t, out[1].t, out[2].t, block=block)
            [b.bits() for b in out]
            got.append([b.raw[b.lo:b.end] for b in out])
        assert torch.equal(got[0][0], src[:n].view(torch.uint8)), n
        for other in got[1:]:
            for a, b in zip(got[0], other):
                assert torch.equal(a, b), n


def random_copies(n, k, grad_block, gen):
    """k int4 copies of n elements, each with codes of its own and scales of
    its own per block, and the gradient that they sum to.  The sum is the fma
    chain of the method bit for bit: with scales within 1e-5 .. 2e-4 a partial
    sum and a product together span fewer than 53 bits, so each sum in 64 bits
    is exact and rounds to 32 once."""
    codes, scales, acc = [], [], torch.zeros(n, device="cuda")
    nb = -(-n // grad_block)
    for _ in range(k):
        c = torch.randint(0, 256, ((n + 1) // 2,), dtype=torch.uint8, device="cuda", generator=gen)
        s = torch.empty(nb, device="cuda").uniform_(1e-5, 2e-4, generator=gen)
        x = torch.stack((c & 0xF, c >> 4), 1).reshape(-1)[:n].to(torch.int8)
        x = ((x ^ 8) - 8).double()
        x *= s.repeat_interleave(grad_block)[:n].double()
        acc = (acc.double() + x).float()
        codes.append(c)
        scales.append(s)
    return codes, scales, acc * torch.tensor(1.0 / k, dtype=torch.float32, device="cuda")


def interleaved(codes, scales, n, grad_block, offset):
    """Those copies in one receive buffer, its codes `offset` bytes into it."""
    k, nb, half = len(codes), -(-n // grad_block), grad_block // 2
    c = torch.zeros(offset + nb * k * half, dtype=torch.uint8, device="cuda")
    for q in range(k):
        flat = torch.zeros(nb * half, dtype=torch.uint8, device="cuda")
        flat[:codes[q].numel()] = codes[q]
        c[offset:].view(nb, k, half)[:, q] = flat.view(nb, half)
    return c[offset:], torch.stack(scales, 1).reshape(-1)


NAMES7 = NAMES + ("codes", "scales")


def check_pass(zpp, n, block, layout, k, grad_block, adamw=True, offset=0, secondary=True):
    """The step with its copies and codes in one call, the receive step and the
    reduction, against the gradient itself through the step and the refresh with
    its quantization as calls of their own, bit for bit."""
    gen = torch.Generator(device="cuda").manual_seed(n * 64 + k)
    p = torch.empty(n, device="cuda").normal_(0, 0.02, generator=gen)
    if layout == "gradient":
        g = torch.empty(n, device="cuda").normal_(0, 1e-3, generator=gen)
    else:
        codes, scales, g = random_copies(n, k, grad_block, gen)
    hp, kw = dict(HP, step=3, adamw=adamw), dict(scale_out=float(np.float32(1.0 / k)))

    def state():
        st = [Buf(n, torch.float32, offset) for _ in range(3)] + [Buf(n, torch.int16, offset)]
        for b, x in zip(st, (p, g * 0.5, g * g)):
            b.t.copy_(x)
        return st

    def outputs():
        return [Buf(n, torch.int16, offset), Buf(n, torch.int8, offset),
                Buf(-(-n // block), torch.float32)]

    def same(got, ref, what):
        for x, y, name in zip(got, ref, NAMES7):
            assert x is None or torch.equal(x.raw, y.raw), (what, name)

    ref, ref_out = state(), outputs()
    gb = Buf(n, torch.float32, offset)
    gb.t.copy_(g)
    zpp.adam_partition_step(*[b.t for b in ref[:3]], gb.t, ref[3].t, **hp)
    zpp.refresh_quantize_i8(ref_out[0].t, ref[3].t, ref_out[1].t, ref_out[2].t, block=block)
    got, out = state(), outputs()
    a, o = [b.t for b in got], [b.t for b in out]
    if not secondary:
        out[0] = o[0] = None
    if layout == "gradient":
        zpp.adam_step_refresh_quantize(*a[:3], gb.t, a[3], *o, block=block, **hp)
        return same(got + out, ref + ref_out, "fused")
    if layout == "interleaved":
        src = interleaved(codes, scales, n, grad_block, offset) + (k,)
        calls = (zpp.qgz_receive_step_refresh_quantize_interleaved,
                 zpp.qgz_receive_adam_step_interleaved, zpp.dequant_reduce_i4_interleaved)
    else:
        src = ([torch.cat((c[:offset], c))[offset:] for c in codes], scales)
        calls = (zpp.qgz_receive_step_refresh_quantize, zpp.qgz_receive_adam_step,
                 zpp.dequant_reduce_i4)
    calls[0](*a[:3], *src, a[3], *o, grad_block=grad_block, block=block, **kw, **hp)
    same(got + out, ref + ref_out, "pass")
    got = state()
    a = [b.t for b in got]
    calls[1](*a[:3], *src, a[3], block=grad_block, **kw, **hp)
    same(got, ref, "step")
    r = Buf(n, torch.float32, offset)
    calls[2](*src, n, r.t, block=grad_block, **kw)
    assert torch.equal(r.raw, gb.raw), "reduction"


@pytest.mark.parametrize("sources", [0, 16], ids=["gradient", "receive"])
@pytest.mark.parametrize("block", [192, 320, 832, 1024, 1280, 1344, 2048, 4096])
def test_fused_block_routes(zpp, block, sources):
    """The fused step for blocks other than 64, 128, 256 and 512 at ragged
    lengths and around 8 M elements, where most blocks change from a workgroup
    per block to two kernels; the receive with 16 separate copies."""
    limit = 8 << 20
    for n in (1, block - 1, block, 5 * block + 3, limit, limit + block + 5):
        check_pass(zpp, n, block, "separate" if sources else "gradient", max(sources, 1), 256)


@pytest.mark.parametrize("block", [64, 128, 192, 256, 512, 1024])
def test_fused_with_l2_decay(zpp, block):
    for offset in (0, 3):
        check_pass(zpp, 5 * 4096 + 1029, block, "gradient", 1, 256, adamw=False, offset=offset)


@pytest.mark.parametrize("layout", ["separate", "interleaved"])
@pytest.mark.parametrize("adamw", [True, False], ids=["adamw", "l2"])
@pytest.mark.parametrize("k,grad_block,offset", [(16, 256, 0), (19, 512, 3), (33, 1024, 1),
                                                 (64, 256, 4), (8, 256, 0), (12, 192, 1),
                                                 (17, 320, 0), (24, 64, 5)])
def test_receives(zpp, layout, adamw, k, grad_block, offset):
    """Every int8 block's kernel with few and many int4 copies: whole tiles, a
    partial one, on and off alignment, both forms of the decay.  (Many copies
    take the many-source form with int4 blocks that are multiples of 256.)"""
    for block in (64, 128, 256, 512, 192, 832, 1024, 4096):
        check_pass(zpp, 5 * 4096 + 1029, block, layout, k, grad_block, adamw, offset,
                   secondary=block != 512)


@pytest.mark.parametrize("offset", [0, 1, 3, 4])
@pytest.mark.parametrize("layout,k,block,adamw,secondary", [
    ("gradient", 1, 192, True, True), ("gradient", 1, 2048, False, True),
    ("gradient", 1, 4096, True, False),
    ("separate", 3, 192, True, True), ("separate", 8, 2048, False, True),
    ("separate", 19, 320, True, True), ("separate", 16, 4096, False, False),
    ("interleaved", 1, 2048, False, True), ("interleaved", 8, 192, True, False),
    ("interleaved", 12, 4096, True, True), ("interleaved", 17, 2048, True, True),
    ("interleaved", 16, 320, False, True)])
def test_two_kernels(zpp, layout, k, block, adamw, secondary, offset):
    """Beyond 8 M elements, the step with its copies and then the quantizer over
    the primary it wrote: each source of the gradient, few and many copies, on
    and off alignment."""
    check_pass(zpp, (8 << 20) + 2 * block + 5, block, layout, k, 256, adamw, offset, secondary)


@pytest.mark.parametrize("layout,k,grad_block,block,limit", [
    ("gradient", 1, 256, 832, 24 << 20), ("gradient", 1, 256, 1280, 24 << 20),
    ("gradient", 1, 256, 1024, 104 << 20), ("gradient", 1, 256, 1152, 104 << 20),
    ("separate", 8, 256, 1024, 4 << 20), ("separate", 3, 256, 832, 16 << 20),
    ("separate", 64, 256, 1088, 2 << 20), ("interleaved", 8, 192, 1280, 4 << 20),
    ("interleaved", 4, 256, 1088, 64 << 20), ("interleaved", 9, 256, 960, 16 << 20),
    ("interleaved", 20, 256, 2048, 4 << 20), ("interleaved", 40, 512, 4096, 4 << 20),
    ("separate", 16, 256, 256, 12 << 20), ("separate", 20, 512, 512, 12 << 20),
    ("interleaved", 16, 256, 64, 12 << 20), ("interleaved", 16, 64, 256, 8 << 20),
    ("separate", 20, 1024, 2048, 12 << 20)])
def test_lengths_of_the_rules(zpp, layout, k, grad_block, block, limit):
    """Around the lengths where the number of kernels or the workgroups per CU
    change."""
    for n in (limit, limit + block + 3):
        check_pass(zpp, n, block, layout, k, grad_block)


@pytest.mark.parametrize("block", [64, 128, 256, 1024, 2048, 4096])
def test_i4_slots_by_length(zpp, block):
    """A sender's codes and scales in an interleaved buffer at the lengths where
    the quantizer changes the tiles a wave keeps in flight or caps residency:
    those of the plain layout, at the slots' places, and the other senders' slots
    as they were."""
    k, source = 3, 1
    lengths = ((8, 13, 97) if block <= 256 else (8, 48))
    for n in [(m << 20) + 771 for m in lengths]:
        nb = -(-n // block)
        gen = torch.Generator(device="cuda").manual_seed(n)
        x = torch.empty(n, device="cuda").normal_(0, 1e-3, generator=gen)
        c, s = (torch.zeros(nb * block // 2, dtype=torch.uint8, device="cuda"),
                torch.zeros(nb, device="cuda"))
        zpp.quantize_blockwise_i4(x, c, s, block=block)
        nc, ns = zpp.interleaved_sizes(n, block, k)
        ci = torch.full((nc,), 0x5A, dtype=torch.uint8, device="cuda")
        si = torch.full((ns,), -1.0, device="cuda")
        zpp.quantize_blockwise_i4_interleaved(x, ci, si, source=source, num_src=k, block=block)
        ci, si = ci.view(nb, k, block // 2), si.view(nb, k)
        used = (n + 1) // 2 - (nb - 1) * (block // 2)  # bytes of the last block that hold codes
        assert torch.equal(ci[:-1, source], c.view(nb, -1)[:-1]), n
        assert torch.equal(ci[-1, source, :used], c.view(nb, -1)[-1, :used]), n
        assert torch.equal(si[:, source], s), n
        for q in range(k):
            if q != source:
                assert (ci[:, q] == 0x5A).all() and (si[:, q] == -1.0).all(), (n, q)
        assert (ci[-1, source, used:] == 0x5A).all(), n


@pytest.mark.parametrize("block", [64, 256, 512, 4096])
def test_quantizer_edges(zpp, block):
    """The quantizers at lengths around their whole tiles (rows of 512 elements
    or of one block per wave): what a longer call over whole tiles gives, its
    elements past the end zero, which no absmax sees."""
    tile = max(512, block) * 8
    full = 4 * tile
    rnd = synth.rng(305, block)
    bf16 = (rnd.standard_normal(full).astype(np.float32).view(np.uint32) >> 16).astype(np.int16)
    f32 = rnd.standard_normal(full).astype(np.float32)
    for n in (tile // 2, tile - 1, tile, tile + 1, tile + block + 3, 2 * tile - 8, 2 * tile + 2):
        got = []
        for m in (n, full):
            h, x = bf16.copy(), f32.copy()
            h[n:], x[n:] = 0, 0
            src16, src32 = Buf(m, torch.int16, 0, h), Buf(m, torch.float32, 0, x)
            nb = -(-m // block)
            second = Buf(m, torch.int16)
            c, s, c2, s2 = (Buf(m, torch.int8), Buf(nb, torch.float32),
                            Buf(m, torch.int8), Buf(nb, torch.float32))
            zpp.quantize_blockwise_i8(src16.t, c.t, s.t, block=block)
            zpp.refresh_quantize_i8(second.t, src16.t, c2.t, s2.t, block=block)
            c4, s4 = Buf((m + 1) // 2, torch.uint8), Buf(nb, torch.float32)
            zpp.quantize_blockwise_i4(src32.t, c4.t, s4.t, block=block)
            got.append([b.bits() for b in (c, s, second, c2, s2, c4, s4)])
        same_start(*got, n, ("codes", "scales", "secondary", "codes with the copy",
                             "scales with the copy", "int4 codes", "int4 scales"))
