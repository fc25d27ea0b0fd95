"""Randomised plan layouts against the oracle: many tensors of random sizes
(empty to a few hundred thousand elements) at random 2-byte offsets inside
shared buffers, random tensor ids, random tile shapes (environment
overrides); every element of every tensor is checked after perturb, swap,
restore and both update roundings, and, over binary32 masters, after
members applied from them and the update into them.  Seeded, so every case
is reproducible."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_17310_amd import esopt, workloads as wl
from parity import to_host, report, assert_parity, perturb_delta, update_delta

pytestmark = pytest.mark.gpu

SHAPES = [(256, 4), (256, 8), (512, 4), (512, 8), (1024, 4), (1024, 8)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("case", range(6))
def test_random_layout(case, monkeypatch):
    rng = np.random.default_rng(1000 + case)
    threads, groups = SHAPES[rng.integers(len(SHAPES))]
    monkeypatch.setenv("ESOPT_THREADS", str(threads))
    monkeypatch.setenv("ESOPT_GROUPS", str(groups))
    n_t = int(rng.integers(1, 25))
    sizes = [int(x) for x in np.where(rng.random(n_t) < 0.15, rng.integers(0, 20, n_t),
                                      rng.integers(1, 300_000, n_t))]
    offsets = [int(x) for x in rng.integers(0, 9, n_t)]      # elements: 0 .. 16 bytes
    ids = [int(x) for x in rng.choice(1 << 20, n_t, replace=False)]
    print("case", case, "shape", threads, groups, "tensors", list(zip(sizes, offsets)))
    host = [wl.random_bf16_bits(n, 7000 + 31 * case + i) for i, n in enumerate(sizes)]
    # all tensors in one device buffer, each at its offset past a 16-byte boundary
    starts, cur = [], 0
    for n, off in zip(sizes, offsets):
        cur = (cur + 7) // 8 * 8 + off
        starts.append(cur)
        cur += n
    buf = torch.zeros(cur + 8, dtype=torch.bfloat16, device="cuda")
    flat = np.zeros(cur + 8, dtype=np.uint16)
    for s, h in zip(starts, host):
        flat[s:s + h.size] = h
    buf.copy_(torch.from_numpy(flat.view(np.int16)).view(torch.bfloat16))
    views = [buf[s:s + n] for s, n in zip(starts, sizes)]
    plan = esopt.Plan(views, tensor_ids=ids)
    seeds = [int(x) for x in rng.integers(0, 1 << 62, 4)]
    signs = [1, -1, 1, 1]
    r = rng.random(4).astype(np.float32)
    sigma, alpha = 1e-3, 5e-4

    def snap():
        torch.cuda.synchronize()
        return [to_host(v) for v in views]
    x0 = snap()
    plan.perturb(seeds[0], 1, sigma)
    x1 = snap()
    plan.swap(seeds[0], 1, seeds[1], -1, sigma)
    x2 = snap()
    plan.restore(seeds[1], -1, sigma)
    x3 = snap()
    plan.update(seeds, signs, torch.from_numpy(r).cuda(), alpha)
    x4 = snap()
    plan.update(seeds, signs, torch.from_numpy(r).cuda(), alpha,
                flags=esopt.ES_UPDATE_STOCHASTIC_ROUND, round_seed=case)
    x5 = snap()
    plan.close()
    # bytes outside the tensors are untouched
    full = to_host(buf)
    mask = np.ones(full.size, bool)
    for s, n in zip(starts, sizes):
        mask[s:s + n] = False
    assert np.all(full[mask] == flat[mask])
    # every element of every tensor, pooled per pass over the case's tensors
    # and held to the parity bar (tests/parity.py: <= 1 ulp on >= 99.99 %,
    # never above 2 ulp, >= 99.9 % bit-exact)
    stages = ("perturb", "swap", "restore", "update", "update_sr")
    pooled = {k: ([], [], [], []) for k in stages}
    for i, (tid, n) in enumerate(zip(ids, sizes)):
        if n == 0:
            continue
        el = np.arange(n, dtype=np.uint64)
        checks = [
            (x1[i], oracle.perturb(x0[i], seeds[0], tid, 1, sigma), x0[i],
             perturb_delta(seeds[0], tid, 1, sigma, el)),
            (x2[i], oracle.swap(x1[i], tid, seeds[0], 1, sigma, seeds[1], -1, sigma), x1[i],
             perturb_delta(seeds[0], tid, -1, sigma, el) + perturb_delta(seeds[1], tid, -1, sigma, el)),
            (x3[i], oracle.restore(x2[i], seeds[1], tid, -1, sigma), x2[i],
             perturb_delta(seeds[1], tid, 1, sigma, el)),
            (x4[i], oracle.update(x3[i], tid, seeds, signs, r, alpha, sigma)[0], x3[i],
             update_delta(tid, seeds, signs, r, alpha, sigma, 0, el)),
            (x5[i], oracle.update(x4[i], tid, seeds, signs, r, alpha, sigma,
                                  flags=esopt.ES_UPDATE_STOCHASTIC_ROUND, round_seed=case)[0],
             x4[i], update_delta(tid, seeds, signs, r, alpha, sigma, 0, el)),
        ]
        for k, parts in zip(stages, checks):
            for acc, part in zip(pooled[k], parts):
                acc.append(part)
    for k in stages:
        got, exp, base, delta = (np.concatenate(a) for a in pooled[k])
        rep = report(got, exp, base, delta)
        print("case", case, k, rep)
        assert_parity(rep, f"case {case} {k}")


@pytest.mark.parametrize("case", range(4))
def test_random_master_layout(case, monkeypatch):
    """Binary32 masters (16-byte aligned, at random gaps in one float32
    buffer) of a random bf16 layout: a member applied from them, the update
    into them and a member applied from the updated masters, every element
    against the oracle (the bf16 values at the parity bar, the masters within
    the bound of the kernel's arithmetic, the bf16 copy after the update the
    rounding of the GPU's masters), and no byte outside the tensors or the
    masters written."""
    from parity import assert_master_parity, master_report, master_tolerance
    rng = np.random.default_rng(3000 + case)
    threads, groups = SHAPES[rng.integers(len(SHAPES))]
    monkeypatch.setenv("ESOPT_THREADS", str(threads))
    monkeypatch.setenv("ESOPT_GROUPS", str(groups))
    n_t = int(rng.integers(1, 17))
    sizes = [int(x) for x in np.where(rng.random(n_t) < 0.15, rng.integers(0, 20, n_t),
                                      rng.integers(1, 300_000, n_t))]
    offsets = [int(x) for x in rng.integers(0, 9, n_t)]
    ids = [int(x) for x in rng.choice(1 << 20, n_t, replace=False)]
    print("case", case, "shape", threads, groups, "tensors", list(zip(sizes, offsets)))
    starts, cur = [], 0
    for n, off in zip(sizes, offsets):
        cur = (cur + 7) // 8 * 8 + off
        starts.append(cur)
        cur += n
    buf = torch.zeros(cur + 8, dtype=torch.bfloat16, device="cuda")
    views = [buf[s:s + n] for s, n in zip(starts, sizes)]
    mstarts, mcur = [], 0
    for n in sizes:                                   # 16-byte aligned, random gaps
        mcur = (mcur + 3) // 4 * 4 + 4 * int(rng.integers(0, 3))
        mstarts.append(mcur)
        mcur += n
    m0 = [(rng.standard_normal(n) * 0.02).astype(np.float32) for n in sizes]
    mflat = np.full(mcur + 4, 7.0, np.float32)        # sentinel outside the masters
    for s, m in zip(mstarts, m0):
        mflat[s:s + m.size] = m
    mbuf = torch.from_numpy(mflat).cuda()
    mviews = [mbuf[s:s + n] for s, n in zip(mstarts, sizes)]
    plan = esopt.Plan(views, tensor_ids=ids)
    plan.set_master(mviews)
    seeds = [int(x) for x in rng.integers(0, 1 << 62, 4)]
    signs = [1, -1, 1, 1]
    r = rng.random(4).astype(np.float32)
    sigma, alpha = 1e-3, 5e-4

    def snap():
        torch.cuda.synchronize()
        return [to_host(v) for v in views], [m.cpu().numpy() for m in mviews]
    plan.perturb_master(seeds[0], 1, sigma)
    x1, _ = snap()
    plan.update(seeds, signs, torch.from_numpy(r).cuda(), alpha, flags=esopt.ES_UPDATE_MASTER)
    x2, m2 = snap()
    plan.perturb_master(seeds[1], -1, 2 * sigma)
    x3, m3 = snap()
    plan.close()
    full = mbuf.cpu().numpy()
    mask = np.ones(full.size, bool)
    for s, n in zip(mstarts, sizes):
        mask[s:s + n] = False
    assert np.all(full[mask] == 7.0)
    fb = to_host(buf)
    bmask = np.ones(fb.size, bool)
    for s, n in zip(starts, sizes):
        bmask[s:s + n] = False
    assert np.all(fb[bmask] == 0)

    z, _ = oracle.zscore(r)
    c = oracle.update_coefficient(alpha, sigma, len(seeds), 0)
    d, w = oracle.member_weights(seeds, signs, z, c)
    live = [(sd, wd) for sd, wd in zip(d, w) if wd != 0.0]

    def rne(m):
        return oracle.f64_to_bf16_rne(np.asarray(m, np.float32).astype(np.float64))
    pooled = {k: ([], [], [], []) for k in ("apply", "apply after update")}
    mrep = ([], [], [])
    for i, (tid, n) in enumerate(zip(ids, sizes)):
        if n == 0:
            continue
        el = np.arange(n, dtype=np.uint64)
        for k, got, mm, sd, sg, sg_sigma in (("apply", x1[i], m0[i], seeds[0], 1, sigma),
                                             ("apply after update", x3[i], m2[i], seeds[1], -1,
                                              2 * sigma)):
            for acc, part in zip(pooled[k], (got, oracle.perturb_master(mm, sd, tid, sg, sg_sigma),
                                             rne(mm), perturb_delta(sd, tid, sg, sg_sigma, el))):
                acc.append(part)
        exp, _, st = oracle.update_master(m0[i], tid, seeds, signs, r, alpha, sigma)
        assert st == 0
        for acc, part in zip(mrep, (m2[i], exp, master_tolerance(exp, live, tid, el))):
            acc.append(part)
        np.testing.assert_array_equal(x2[i], rne(m2[i]))          # the copy: the masters' rounding
        np.testing.assert_array_equal(m3[i], m2[i])               # applying leaves the masters
    for k, parts in pooled.items():
        rep = report(*(np.concatenate(a) for a in parts))
        print("case", case, k, rep)
        assert_parity(rep, f"case {case} {k}")
    rep = master_report(*(np.concatenate(a) for a in mrep))
    print("case", case, "masters", rep)
    assert_master_parity(rep, f"case {case} masters")


@pytest.mark.parametrize("case", range(4))
def test_random_int8_layout(case, monkeypatch):
    from parity import q_tolerance, qreport, assert_qparity
    rng = np.random.default_rng(2000 + case)
    threads, groups = SHAPES[rng.integers(len(SHAPES))]
    monkeypatch.setenv("ESOPT_THREADS", str(threads))
    monkeypatch.setenv("ESOPT_QGROUPS", str(groups))
    n_t = int(rng.integers(1, 16))
    sizes = [int(x) for x in rng.integers(1, 400_000, n_t)]
    rows = [int(rng.choice([0, 8, 24, 64, 1024, 5120])) for _ in range(n_t)]
    offsets = [int(x) for x in rng.integers(0, 17, n_t)]     # bytes
    ids = [int(x) for x in rng.choice(1 << 20, n_t, replace=False)]
    print("case", case, "shape", threads, groups, list(zip(sizes, rows, offsets)))
    codes = [rng.integers(-127, 128, n).astype(np.int8) for n in sizes]
    scales = [rng.uniform(2e-4, 1e-3, 1 if r == 0 else -(-n // r)).astype(np.float32)
              for n, r in zip(sizes, rows)]
    for sc in scales:
        if sc.size > 4:
            sc[int(rng.integers(sc.size))] = 0.0                 # an invalid row
    starts, cur = [], 0
    for n, off in zip(sizes, offsets):
        cur = (cur + 15) // 16 * 16 + off
        starts.append(cur)
        cur += n
    flat = np.zeros(cur + 16, np.int8)
    for s, c in zip(starts, codes):
        flat[s:s + c.size] = c
    buf = torch.from_numpy(flat).cuda()
    views = [buf[s:s + n] for s, n in zip(starts, sizes)]
    sdev = [torch.from_numpy(sc).cuda() for sc in scales]
    plan = esopt.QPlan(views, sdev, rows, tensor_ids=ids)
    seeds = [int(x) for x in rng.integers(0, 1 << 62, 3)]
    r = rng.random(3).astype(np.float32)

    def snap():
        torch.cuda.synchronize()
        return [v.cpu().numpy().copy() for v in views]
    q0 = snap()
    plan.perturb(seeds[0], -1, 1e-3)
    q1 = snap()
    plan.restore(seeds[0], -1, 1e-3)
    q2 = snap()
    plan.update(seeds, [1, 1, 1], torch.from_numpy(r).cuda(), 5e-3, round_seed=case)
    q3 = snap()
    plan.close()
    full = buf.cpu().numpy()
    mask = np.ones(full.size, bool)
    for s, n in zip(starts, sizes):
        mask[s:s + n] = False
    assert np.all(full[mask] == flat[mask])
    for i, (tid, n, row, sc) in enumerate(zip(ids, sizes, rows, scales)):
        el = np.arange(n, dtype=np.uint64)
        d, rr, ok = oracle.offset_values(sc, row, seeds[0], tid, -1, 1e-3, el)
        s = np.where(ok, oracle.row_scales(sc, row, el), 1.0)
        eps = oracle.normals(seeds[0], tid, el)
        tol = q_tolerance(float(np.float32(1e-3)) / s, np.abs(float(np.float32(1e-3)) * eps) / s, d)
        v = d + (2 * rr + 1) * 2.0 ** -10
        assert_qparity(qreport(q1[i], q0[i], v, tol, ok), f"case {case} tensor {i} perturb")
        assert_qparity(qreport(q2[i], q1[i], v, tol, ok, negate=True), f"case {case} tensor {i} restore")
        d, rr, ok, live, st = oracle.update_values(sc, row, tid, seeds, [1, 1, 1], r, 5e-3, 0.0,
                                                   elems=el, round_seed=case)
        wsum = np.zeros(n)
        nsum = np.zeros(n)
        for sd, w in live:
            wsum += abs(w) / s
            nsum += np.abs(w * oracle.normals(sd, tid, el)) / s
        v = d + rr * 2.0 ** -16
        assert_qparity(qreport(q3[i], q2[i], v, q_tolerance(wsum, nsum, d), ok),
                       f"case {case} tensor {i} update")


def test_many_tiny_tensors():
    """20 000 tensors of 1-200 elements at random 2-byte offsets (a tile per
    tensor, most of them tails): the galloping tile-to-tensor lookup; 400
    tensors checked element by element after perturb and update, and every
    byte between tensors untouched."""
    rng = np.random.default_rng(77)
    n_t = 20000
    sizes = rng.integers(1, 201, n_t)
    offsets = rng.integers(0, 9, n_t)
    starts, cur = [], 0
    for n, off in zip(sizes, offsets):
        cur = (cur + 7) // 8 * 8 + int(off)
        starts.append(cur)
        cur += int(n)
    flat = wl.random_bf16_bits(cur + 8, 78)
    buf = torch.from_numpy(flat.view(np.int16)).view(torch.bfloat16).cuda()
    views = [buf[s:s + int(n)] for s, n in zip(starts, sizes)]
    plan = esopt.Plan(views)
    r = rng.random(5).astype(np.float32)
    plan.perturb(9, -1, 1e-3)
    torch.cuda.synchronize()
    mid = to_host(buf)
    plan.update([1, 2, 3, 4, 5], [1] * 5, torch.from_numpy(r).cuda(), 5e-4)
    torch.cuda.synchronize()
    out = to_host(buf)
    plan.close()
    mask = np.ones(flat.size, bool)
    for s, n in zip(starts, sizes):
        mask[s:s + int(n)] = False
    assert np.all(out[mask] == flat[mask])
    pooled = {"perturb": ([], [], [], []), "update": ([], [], [], [])}
    for i in rng.choice(n_t, 400, replace=False):
        s, n = starts[i], int(sizes[i])
        el = np.arange(n, dtype=np.uint64)
        exp_u, _ = oracle.update(mid[s:s + n], int(i), [1, 2, 3, 4, 5], [1] * 5, r, 5e-4, 1e-3)
        for k, parts in (("perturb", (mid[s:s + n], oracle.perturb(flat[s:s + n], 9, int(i), -1, 1e-3),
                                      flat[s:s + n], perturb_delta(9, int(i), -1, 1e-3, el))),
                         ("update", (out[s:s + n], exp_u, mid[s:s + n],
                                     update_delta(int(i), [1, 2, 3, 4, 5], [1] * 5, r, 5e-4, 1e-3, 0,
                                                  el)))):
            for acc, part in zip(pooled[k], parts):
                acc.append(part)
    for k, parts in pooled.items():
        rep = report(*(np.concatenate(a) for a in parts))
        print("many tiny tensors", k, rep)
        assert_parity(rep, f"many tiny tensors {k}")
        assert rep["max_ulp"] <= 1.0, (k, rep)


def test_many_tiny_int8_tensors():
    from parity import q_tolerance, qreport, assert_qparity
    rng = np.random.default_rng(79)
    n_t = 20000
    sizes = rng.integers(1, 300, n_t)
    starts, cur = [], 0
    for n in sizes:
        cur = (cur + 15) // 16 * 16 + int(rng.integers(0, 17))
        starts.append(cur)
        cur += int(n)
    flat = rng.integers(-127, 128, cur + 16).astype(np.int8)
    buf = torch.from_numpy(flat).cuda()
    sc = torch.full((1,), 6e-4, device="cuda")
    views = [buf[s:s + int(n)] for s, n in zip(starts, sizes)]
    plan = esopt.QPlan(views, [sc] * n_t, [0] * n_t)
    plan.perturb(4, 1, 1e-3)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    plan.close()
    for i in rng.choice(n_t, 300, replace=False):
        s, n = starts[i], int(sizes[i])
        el = np.arange(n, dtype=np.uint64)
        d, rr, ok = oracle.offset_values([6e-4], 0, 4, int(i), 1, 1e-3, el)
        eps = oracle.normals(4, int(i), el)
        s32 = float(np.float32(1e-3)) / float(np.float32(6e-4))
        tol = q_tolerance(np.full(n, s32), np.abs(s32 * eps), d)
        assert_qparity(qreport(out[s:s + n], flat[s:s + n], d + (2 * rr + 1) * 2.0 ** -10, tol, ok),
                       f"tiny int8 tensor {i}")
