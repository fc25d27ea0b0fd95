"""Tensors whose sizes sit at the edges of the step kernels' cuts (a lane's
8-element groups, a workgroup's step of 4096 or 8192 elements, the 65
536-element tile), at bases that are 16-byte aligned and not: the update in
its forms, perturb, swap and a member applied from masters against the oracle,
the bytes around each tensor untouched, and a plan of so many tiny tensors
that its tail tiles are not cut into steps."""
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
    """Above 65 536 tail tiles the tail items are whole tiles, whose longest
    then takes sixteen steps."""
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
