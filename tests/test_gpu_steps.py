"""Tensors whose sizes sit at the edges of the step kernels' cuts (a lane's
8-element groups, a workgroup's step of 4096 or 8192 elements, the 65
536-element tile), at bases that are 16-byte aligned and not: the update in
its forms, perturb, swap and a member applied from masters against the oracle,
the bytes around each tensor untouched, and a plan of very many tiny tensors
and a long one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_17310_amd import esopt, workloads as wl
from parity import (to_device, to_host, report, assert_parity, update_delta, perturb_delta)

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 8, 9, 2047, 2048, 2049, 4095, 4096, 4097, 16384 + 5, 65536, 65536 * 2 + 4099]
SEEDS, SIGNS, ALPHA, SIGMA = [11, 12, 13, 11], [1, -1, 1, 1], 5e-4, 1e-3
REWARDS = np.array([0.9, 0.25, 0.5, 0.1], dtype=np.float32)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _buffer(pad, seed=900):
    """All sizes in one buffer, each `pad` elements past a 256-byte boundary
    and followed by at least 8 guard elements."""
    offs, cur = [], 0
    for n in SIZES:
        offs.append(cur + pad)
        cur += -(-(pad + n + 8) // 128) * 128
    bits = wl.random_bf16_bits(cur, seed + pad)
    flat = to_device(bits)
    return bits, flat, [(o, flat[o:o + n]) for o, n in zip(offs, SIZES)]


def _check(bits, flat, parts, expected, delta, what):
    """expected(bits, id) and delta(id, elements) per tensor, one parity bar
    over all of them; everything between the tensors unchanged."""
    got = to_host(flat)
    inside = np.zeros(got.size, dtype=bool)
    pooled = ([], [], [], [])
    for i, (o, t) in enumerate(parts):
        n = t.numel()
        inside[o:o + n] = True
        el = np.arange(n, dtype=np.uint64)
        for acc, part in zip(pooled, (got[o:o + n], expected(bits[o:o + n], i), bits[o:o + n],
                                      delta(i, el))):
            acc.append(part)
    assert np.array_equal(got[~inside], bits[~inside]), f"{what}: values outside the tensors"
    assert_parity(report(*(np.concatenate(p) for p in pooled)), what)


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("flags", [0, esopt.ES_UPDATE_STOCHASTIC_ROUND])
def test_update_at_the_edges(pad, flags):
    bits, flat, parts = _buffer(pad)
    with esopt.Plan([t for _, t in parts]) as plan:
        plan.update(SEEDS, SIGNS, torch.from_numpy(REWARDS).cuda(), ALPHA, flags=flags,
                    round_seed=3)
        torch.cuda.synchronize()
    _check(bits, flat, parts,
           lambda b, i: oracle.update(b, i, SEEDS, SIGNS, REWARDS, ALPHA, SIGMA, flags=flags,
                                      round_seed=3)[0],
           lambda i, el: update_delta(i, SEEDS, SIGNS, REWARDS, ALPHA, SIGMA, flags, el),
           f"update pad {pad} flags {flags}")


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("filler", [0, 17_000_000])
def test_perturbation_passes_at_the_edges(pad, filler):
    """perturb, two-key swap and perturb_master; with a 17 M-element tensor in
    the plan the steps take four groups per lane instead of two."""
    bits, flat, parts = _buffer(pad)
    views = [t for _, t in parts]
    fill_bits = wl.random_bf16_bits(filler + 3, 55) if filler else None
    if filler:
        fill = to_device(fill_bits)
        views.append(fill)
        at = np.concatenate([np.arange(9000), 8 * np.random.default_rng(3).integers(0, filler // 8, 500),
                             np.arange(filler - 9000, filler + 3)]).astype(np.uint64)
    with esopt.Plan(views) as plan:
        def check(call, expected, delta, what):
            before, fbefore = to_host(flat), to_host(fill) if filler else None
            call()
            torch.cuda.synchronize()
            _check(before, flat, parts, lambda b, i: expected(b, i, None), delta, what)
            if filler:
                i = len(parts)
                rep = report(to_host(fill)[at], expected(fbefore[at], i, at), fbefore[at],
                             delta(i, at))
                assert_parity(rep, what + " filler")

        check(lambda: plan.perturb(5, -1, SIGMA),
              lambda b, i, el: oracle.perturb(b, 5, i, -1, SIGMA, elems=el),
              lambda i, el: perturb_delta(5, i, -1, SIGMA, el), "perturb")
        check(lambda: plan.swap(5, -1, 6, 1, SIGMA),
              lambda b, i, el: oracle.swap(b, i, 5, -1, SIGMA, 6, 1, SIGMA, elems=el),
              lambda i, el: perturb_delta(6, i, 1, SIGMA, el), "swap")
        ms = [t.float() for t in views]
        mh = [m.cpu().numpy() for m in ms]
        plan.set_master(ms)
        check(lambda: plan.perturb_master(7, 1, SIGMA),
              lambda b, i, el: oracle.perturb_master(mh[i] if el is None else mh[i][at], 7, i, 1,
                                                     SIGMA, elems=el),
              lambda i, el: perturb_delta(7, i, 1, SIGMA, el), "perturb_master")
    tail = to_host(flat)
    for o, t in parts:
        tail[o:o + t.numel()] = bits[o:o + t.numel()]
    assert np.array_equal(tail, bits)


@pytest.mark.parametrize("pad", [0, 1])
def test_restore_update_and_masters_at_the_edges(pad):
    """One pass against the two it replaces, and the update into masters
    against the plain update of bf16-representable masters, bit for bit."""
    r = torch.from_numpy(REWARDS).cuda()
    outs = []
    for form in ("fused", "apart", "masters"):
        bits, flat, parts = _buffer(pad)
        with esopt.Plan([t for _, t in parts]) as plan:
            if form == "fused":
                plan.restore_update(12, -1, SIGMA, SEEDS, SIGNS, r, ALPHA)
            else:
                plan.restore(12, -1, SIGMA)
            if form == "apart":
                plan.update(SEEDS, SIGNS, r, ALPHA)
            elif form == "masters":
                ms = [t.float() for _, t in parts]
                plan.set_master(ms)
                plan.update(SEEDS, SIGNS, r, ALPHA, flags=esopt.ES_UPDATE_MASTER)
            torch.cuda.synchronize()
        outs.append(to_host(flat))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[1], outs[2])


def test_many_tiny_tensors_and_a_long_one():
    """Tail tiles of one step each, among them two of several: each step's
    workgroup finds its tile."""
    n_tiny, big = 66_000, 150_001
    bits = wl.random_bf16_bits(8 * n_tiny + big, 77)
    flat = to_device(bits)
    views = [flat[8 * i:8 * i + 3] for i in range(n_tiny)] + [flat[8 * n_tiny:]]
    with esopt.Plan(views) as plan:
        plan.update(SEEDS, SIGNS, torch.from_numpy(REWARDS).cuda(), ALPHA)
        torch.cuda.synchronize()
    got = to_host(flat)
    assert np.array_equal(got[:8 * n_tiny].reshape(-1, 8)[:, 3:],
                          bits[:8 * n_tiny].reshape(-1, 8)[:, 3:])
    pooled = ([], [], [], [])
    for i in [0, 1, 255, 8191, 8192, 65_535, n_tiny - 1, n_tiny]:
        o, n = 8 * i, (big if i == n_tiny else 3)
        exp = oracle.update(bits[o:o + n], i, SEEDS, SIGNS, REWARDS, ALPHA, SIGMA)[0]
        d = update_delta(i, SEEDS, SIGNS, REWARDS, ALPHA, SIGMA, 0, np.arange(n, dtype=np.uint64))
        for acc, part in zip(pooled, (got[o:o + n], exp, bits[o:o + n], d)):
            acc.append(part)
    assert_parity(report(*(np.concatenate(p) for p in pooled)), "many tiny tensors")


# ------------------------------------------------------------ quantized plans --
# The GPU's binary32 step is within about 1e-6 of its size of the oracle's, so
# a code differs only where the step lands that close to a rounding threshold:
# a few codes in 1e6 at these steps (a few quanta), by one code.

QSIZES = [1, 15, 16, 17, 4095, 4096, 4097, 32768 + 3, 65536, 65536 + 4096 + 1]


def _qbuffer(fmt, pad, sizes):
    rng = np.random.default_rng(400 + pad)
    offs, cur = [], 0
    for n in sizes:
        offs.append(cur + pad)
        cur += -(-(pad + n + 16) // 256) * 256
    codes = (rng.integers(-127, 128, cur).astype(np.int8) if fmt == "int8"
             else (rng.integers(0, 2, cur) * 128 + rng.integers(0, 127, cur)).astype(np.uint8))
    flat = torch.from_numpy(codes).cuda()
    rows = [8 * (1 + i % 5) if i % 2 else 0 for i in range(len(sizes))]
    scales = [rng.uniform(4e-4, 9e-4, 1 if r == 0 else -(-n // r)).astype(np.float32)
              for r, n in zip(rows, sizes)]
    return codes, flat, offs, rows, scales


def _qexpected(fmt, kind, b, i, row, scales):
    if kind == "update":
        f = oracle.qupdate if fmt == "int8" else oracle.f8update
        return f(b, scales, row, i, SEEDS, SIGNS, REWARDS, 5e-3, SIGMA, round_seed=9)[0]
    perturb, restore = ((oracle.qperturb, oracle.qrestore) if fmt == "int8"
                        else (oracle.f8perturb, oracle.f8restore))
    if kind == "swap":
        b = restore(b, scales, row, 4, i, 1, SIGMA)
    return perturb(b, scales, row, 5, i, 1, SIGMA)


def _qrun(plan, kind):
    if kind == "update":
        plan.update(SEEDS, SIGNS, torch.from_numpy(REWARDS).cuda(), 5e-3, round_seed=9)
    elif kind == "swap":
        plan.swap(4, 1, 5, 1, SIGMA)
    else:
        plan.perturb(5, 1, SIGMA)
    torch.cuda.synchronize()


@pytest.mark.parametrize("fmt", ["int8", "e4m3"])
@pytest.mark.parametrize("kind", ["perturb", "swap", "update"])
@pytest.mark.parametrize("pad", [0, 5])
def test_quantized_passes_at_the_edges(fmt, kind, pad):
    codes, flat, offs, rows, scales = _qbuffer(fmt, pad, QSIZES)
    views = [flat[o:o + n] for o, n in zip(offs, QSIZES)]
    with esopt.QPlan(views, [torch.from_numpy(s).cuda() for s in scales], rows,
                     format=fmt) as plan:
        _qrun(plan, kind)
    got, want = flat.cpu().numpy(), codes.copy()
    for i, (o, n) in enumerate(zip(offs, QSIZES)):
        want[o:o + n] = _qexpected(fmt, kind, codes[o:o + n], i, rows[i], scales[i])
    assert np.mean(got != want) <= 5e-5, np.mean(got != want)
    near = got != want
    assert np.all(np.abs(got[near].astype(int) - want[near].astype(int)) <= 1)
    assert np.mean(got != codes) > 0.3


@pytest.mark.parametrize("n_tensors", [1, 64, 65, 5000])
def test_quantized_lookup_over_many_tensors(n_tensors):
    """The tensor of a workgroup's tile is found 64 table entries at a time."""
    sizes = [33 + 16 * (i % 3) for i in range(n_tensors - 1)] + [70_001]
    codes, flat, offs, rows, scales = _qbuffer("int8", 0, sizes)
    views = [flat[o:o + n] for o, n in zip(offs, sizes)]
    with esopt.QPlan(views, [torch.from_numpy(s).cuda() for s in scales], rows) as plan:
        _qrun(plan, "perturb")
    got = flat.cpu().numpy()
    for i in sorted({0, 1, 62, 63, 64, 4095, 4096, n_tensors - 2, n_tensors - 1}):
        if 0 <= i < n_tensors:
            o, n = offs[i], sizes[i]
            want = _qexpected("int8", "perturb", codes[o:o + n], i, rows[i], scales[i])
            assert np.mean(got[o:o + n] != want) <= 5e-5, i


@pytest.mark.parametrize("sigma", [1e6, 1e30])
def test_int8_steps_beyond_every_code(sigma):
    """Steps of up to 1e38 quanta and beyond clamp to the end they point to,
    and a restore of them to the other."""
    codes, flat, offs, rows, scales = _qbuffer("int8", 0, [5000])
    s = np.full_like(scales[0], 1e-30 if sigma > 1e20 else 1e-4)
    with esopt.QPlan([flat[:5000]], [torch.from_numpy(s).cuda()], [0]) as plan:
        plan.perturb(3, 1, sigma)
        torch.cuda.synchronize()
        up = flat[:5000].cpu().numpy()
        # every such step saturates, so the signs of smaller ones say where
        want = oracle.qperturb(codes[:5000], np.full_like(s, 1e-4), 0, 3, 0, 1, 1e6)
        assert np.array_equal(up, want) and set(np.unique(np.abs(up))) == {127}
        plan.restore(3, 1, sigma)
        torch.cuda.synchronize()
        assert np.array_equal(flat[:5000].cpu().numpy(), -want)


@pytest.mark.parametrize("fmt", ["int8", "e4m3"])
def test_invalid_scales_keep_their_codes_at_the_largest_sigma(fmt):
    """sigma sqrt(2 ln 2) is beyond binary32 at sigma 3e38; rows whose scale is
    not a normal positive finite value keep every code all the same."""
    rows, n = 64, 6 * 64
    codes = np.arange(n).astype(np.uint8) if fmt == "e4m3" else np.arange(n).astype(np.int8)
    flat = torch.from_numpy(codes).cuda()
    s = np.array([0.0, -1.0, np.inf, np.nan, 1e-40, 1e-3], dtype=np.float32)
    with esopt.QPlan([flat], [torch.from_numpy(s).cuda()], [rows], format=fmt) as plan:
        plan.perturb(3, 1, 3e38)
        plan.swap(3, 1, 4, -1, 3e38)
        plan.restore(4, -1, 3e38)
    torch.cuda.synchronize()
    got = flat.cpu().numpy()
    assert np.array_equal(got[:5 * rows], codes[:5 * rows])
    assert np.mean(got[5 * rows:] != codes[5 * rows:]) > 0.9


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 1024])
def test_populations_at_the_table_limits(n):
    """Up to 128 members the tables travel in the kernel arguments, above that
    through the scratch; seeds repeat out of order, with both signs."""
    rng = np.random.default_rng(n)
    pool = rng.integers(0, 1 << 63, max(1, n // 2))
    seeds = [int(x) for x in rng.choice(pool, n)]
    signs = [int(x) for x in rng.choice([-1, 1], n)]
    r = rng.standard_normal(n).astype(np.float32)
    bits = wl.random_bf16_bits(777, 5)
    t = to_device(bits)
    z = torch.full((n,), float("nan"), device="cuda")
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    flags = esopt.ES_REWARDS_ARE_WEIGHTS if n == 1 else 0
    with esopt.Plan([t]) as plan:
        plan.update(seeds, signs, torch.from_numpy(r).cuda(), ALPHA, flags=flags, z_out=z,
                    status_out=st)
        torch.cuda.synchronize()
    assert int(st.item()) == 0
    np.testing.assert_allclose(z.cpu().numpy(), r if flags else oracle.zscore(r)[0], rtol=1e-6,
                               atol=1e-7)
    exp, _ = oracle.update(bits, 0, seeds, signs, r, ALPHA, SIGMA, flags=flags)
    rep = report(to_host(t), exp, bits,
                 update_delta(0, seeds, signs, r, ALPHA, SIGMA, flags, np.arange(777, dtype=np.uint64)))
    assert_parity(rep, f"population of {n}")


@pytest.mark.parametrize("per_cu", [None, "1"])
def test_checksum_of_a_plan_of_whole_tiles_is_its_parts(per_cu, monkeypatch):
    """40 M elements run whole tiles, one per workgroup or, with a workgroup per
    compute unit, two or three in turn, an eighth of them tiles cut in eighths or
    halves; the parts' checksums add up to the whole's, and the last part's is
    the oracle's."""
    if per_cu is not None:
        monkeypatch.setenv("ESOPT_UPDATE_WG_PER_CU", per_cu)
    n = 40_000_000 + 24
    bits = wl.random_bf16_bits(n, 8)
    t = to_device(bits)
    cuts = [0, 8 * 60_000, 8 * 700_000, 8 * 2_400_000, n - 100_003 - (n - 100_003) % 8, n]
    with esopt.Plan([t], tensor_ids=[3]) as plan:
        whole = plan.checksum()
    total = 0
    for a, b in zip(cuts, cuts[1:]):
        with esopt.Plan([t[a:b]], tensor_ids=[3], offsets=[a]) as part:
            last = part.checksum()
            total += last
    assert whole == total % (1 << 64)
    assert last == oracle.plan_checksum([(bits[cuts[-2]:], 3, cuts[-2])])


def test_every_element_of_many_steps_is_passed_over_once():
    """17 M zeros perturbed once hold sigma times their normals: the steps'
    order over the XCDs leaves none out and takes none twice.  bf16 carries 8
    significant bits, so a nearest-even value is within 2^-8 = 3.91e-3 of what it
    rounds, relatively (an element left out is off by 1, one taken twice too); the
    binary32 products add under 1e-6."""
    n = 17_000_000
    t = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    with esopt.Plan([t], tensor_ids=[6]) as plan:
        plan.perturb(21, 1, SIGMA)
    eps = esopt.normals(21, 6, 0, n)
    torch.cuda.synchronize()
    assert bool(((t.float() - SIGMA * eps).abs() <= 3.92e-3 * SIGMA * eps.abs() + 1e-9).all())


@pytest.mark.parametrize("per_cu", ["1", "8"])
def test_quantized_checksum_of_whole_tiles_is_its_parts(per_cu, monkeypatch):
    """The same for codes (610 tiles of 65 536)."""
    monkeypatch.setenv("ESOPT_UPDATE_WG_PER_CU", per_cu)
    n, s = 40_000_000 + 32, torch.ones(1, device="cuda")
    codes = np.random.default_rng(9).integers(-127, 128, n).astype(np.int8)
    t = torch.from_numpy(codes).cuda()
    cuts = [0, 16 * 30_000, 16 * 900_000, n - 100_003 - (n - 100_003) % 16, n]
    with esopt.QPlan([t], [s], [0], tensor_ids=[3]) as plan:
        whole = plan.checksum()
    total = 0
    for a, b in zip(cuts, cuts[1:]):
        with esopt.QPlan([t[a:b]], [s], [0], tensor_ids=[3], offsets=[a]) as part:
            last = part.checksum()
            total += last
    assert whole == total % (1 << 64)
    assert last == oracle.qchecksum(codes[cuts[-2]:], 3, cuts[-2])


# ---------------------------------------------------- cuts chosen by plan size --
# Groups per lane, the steps' order over the XCDs and the quantized passes' steps
# per workgroup follow from a plan's size, so one large plan is compared with the
# plans of its parts, which are too small for any of them: the same bits.

def test_parts_of_a_plan_hold_the_bits_of_the_whole():
    """20 M elements take four groups per lane in full tiles and runs of steps per
    XCD, a tenth of them two groups and no runs."""
    n, parts = 20_000_003, 10
    cuts = [n * i // parts // 8 * 8 for i in range(parts)] + [n]
    bits = to_device(wl.random_bf16_bits(n, 71))
    master = bits.float() + 1e-5
    r = torch.from_numpy(REWARDS).cuda()

    def run(spans):
        t, m, seen = bits.clone(), master.clone(), []
        plans = [esopt.Plan([t[a:b]], tensor_ids=[9], offsets=[a]) for a, b in spans]
        for i, (p, (a, b)) in enumerate(zip(plans, spans)):
            own = torch.zeros(b - a, device="cuda").copy_(m[a:b])     # 16-byte aligned
            p.set_master([own])
            spans[i] = (a, b, own)

        def each(call):
            for p in plans:
                call(p)
            seen.append(t.clone())
        each(lambda p: p.perturb(5, -1, SIGMA))
        each(lambda p: p.swap(5, -1, 6, 1, SIGMA))
        each(lambda p: p.swap(6, 1, 6, -1, SIGMA))
        each(lambda p: p.stream_pass())
        each(lambda p: p.restore_update(6, -1, SIGMA, [6, 7], [-1, 1], r[:2], ALPHA))
        each(lambda p: p.update(SEEDS, SIGNS, r, ALPHA, flags=esopt.ES_UPDATE_STOCHASTIC_ROUND,
                                round_seed=4))
        each(lambda p: p.perturb_master(8, 1, SIGMA))
        each(lambda p: p.update(SEEDS, SIGNS, r, ALPHA, flags=esopt.ES_UPDATE_MASTER))
        seen.append(torch.cat([own for *_, own in spans]))
        each(lambda p: p.perturb_master(8, 1, 0.0))
        torch.cuda.synchronize()
        for p in plans:
            p.close()
        return seen
    for i, (x, y) in enumerate(zip(run([(0, n)]), run(list(zip(cuts, cuts[1:]))))):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), i


@pytest.mark.parametrize("fmt", ["int8", "e4m3"])
@pytest.mark.parametrize("n", [51_000_000, 101_000_000, 202_000_000])
def test_parts_of_a_quantized_plan_hold_the_codes_of_the_whole(fmt, n):
    """Two, four and eight steps per workgroup against the one of the parts; the
    whole at an odd base too, where all of it is tail steps."""
    row, parts = 64, 5
    n -= n % row
    cuts = [n * i // parts // row * row for i in range(parts)] + [n]
    gen = torch.Generator(device="cuda").manual_seed(n)
    codes = torch.randint(0, 127, (n,), device="cuda", dtype=torch.uint8, generator=gen)
    scales = torch.empty(n // row, device="cuda").uniform_(4e-4, 9e-4, generator=gen)
    r = torch.from_numpy(REWARDS).cuda()

    def run(spans, pad=0):
        buf = torch.zeros(n + 16, dtype=torch.uint8, device="cuda")
        t, seen = buf[pad:pad + n].copy_(codes), []
        v = t if fmt == "e4m3" else t.view(torch.int8)
        plans = [esopt.QPlan([v[a:b]], [scales[a // row:b // row].clone()], [row],
                             tensor_ids=[9], offsets=[a], format=fmt) for a, b in spans]

        def each(call):
            for p in plans:
                call(p)
            seen.append(t.clone())
        each(lambda p: p.perturb(5, -1, SIGMA))
        each(lambda p: p.swap(5, -1, 6, 1, SIGMA))
        each(lambda p: p.restore(6, 1, SIGMA))
        each(lambda p: p.update(SEEDS, SIGNS, r, ALPHA, round_seed=4))
        torch.cuda.synchronize()
        for p in plans:
            p.close()
        return seen
    want = run(list(zip(cuts, cuts[1:])))
    for pad in (0, 3):
        for i, (x, y) in enumerate(zip(run([(0, n)], pad), want)):
            assert torch.equal(x, y), (pad, i)
