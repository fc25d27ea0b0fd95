"""Full-size parameter sets (0.5B, 4B, 27B-shaped; and the 4B set with a
256-member update) in the launch configuration the benchmark times: one
plan over every tensor, one launch per pass.  Outputs are checked on sampled
elements that the oracle recomputes one by one (every element of a
counter-based, elementwise method can be checked in isolation): random
elements of every tensor, each tensor's first and last elements, and both
sides of the tile transitions the plan actually lays out for that tensor
(taken from the library's own tiling, es_tile_layout, at the tensor's
address): the head tail into the first full tile, the first and the last
full-to-full transitions, and the last full tile into the trailing tail, so
that the full-tile path and the bounds-checked tail path are both
sampled where they meet."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_17310_amd import esopt, workloads as wl
from parity import to_host, report, assert_parity, perturb_delta, update_delta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _tile_edges(view):
    """Elements on both sides of the tile transitions of one tensor: every
    tail tile's first and last element (the head tail before the first full
    tile, the trailing tail after the last), the first full tile's first and
    last element, the first full-to-full transition, the last full-to-full
    transition and the last full tile's last element; each with its
    neighbours on both sides."""
    tiles = esopt.tile_layout(view.data_ptr(), view.numel(), 0)
    full = sorted((a, b) for a, b, f, _ in tiles if f)
    tail = [(a, b) for a, b, f, _ in tiles if not f]
    edges = []
    for a, b in tail:
        edges += [a, b - 1]
    if full:
        edges += [full[0][0], full[0][1] - 1, full[-1][0], full[-1][1] - 1]
        if len(full) > 1:
            edges += [full[1][0], full[-2][1] - 1]
    pts = set()
    for e in edges:
        pts.update((e - 1, e, e + 1))
    return [p for p in pts if 0 <= p < view.numel()], len(full), len(tail)


def _samples(view, rng, k=256):
    numel = view.numel()
    edges, n_full, n_tail = _tile_edges(view)
    fixed = [0, 1, 2, 3, 4, 7, 8, numel // 2, numel - 8, numel - 2, numel - 1] + edges
    idx = np.concatenate([np.array([i for i in fixed if 0 <= i < numel], dtype=np.int64),
                          rng.integers(0, numel, size=min(k, numel))])
    return np.unique(idx), n_full, n_tail


def _gather(views, idx_dev):
    return [to_host(v.view(-1).index_select(0, i)) for v, i in zip(views, idx_dev)]


def _run(W, n_members=None, samples_per_tensor=256):
    seeds = W.seeds if n_members is None else tuple(range(n_members))
    signs = W.signs if n_members is None else (1,) * n_members
    rng = np.random.default_rng(7)
    flat, views = wl.device_params(W)
    plan = esopt.Plan(views)
    assert plan.numel == W.n_params
    picked = [_samples(v, rng, samples_per_tensor) for v in views]
    idx = [p[0] for p in picked]
    # the sample covers both kinds of tile where they meet: every tensor with
    # full tiles has its first and last full-tile elements sampled
    assert sum(p[1] for p in picked) > 0 and sum(p[2] for p in picked) > 0
    idx_dev = [torch.from_numpy(i).cuda() for i in idx]
    sigma = W.sigma0
    theta0 = _gather(views, idx_dev)
    seed, sign = seeds[-1], signs[-1]
    plan.perturb(seed, sign, sigma)
    torch.cuda.synchronize()
    pert = _gather(views, idx_dev)
    seed_b, sign_b = seeds[0], signs[0]
    plan.swap(seed, sign, seed_b, sign_b, sigma)
    torch.cuda.synchronize()
    swp = _gather(views, idx_dev)
    plan.restore(seed_b, sign_b, sigma)
    torch.cuda.synchronize()
    rest = _gather(views, idx_dev)
    r = wl.rewards(W, n=len(seeds))
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    plan.update(seeds, signs, torch.from_numpy(r).cuda(), W.alpha, sigma=sigma, status_out=status)
    torch.cuda.synchronize()
    upd = _gather(views, idx_dev)
    assert int(status.item()) == 0
    sr_flags, round_seed = esopt.ES_UPDATE_STOCHASTIC_ROUND, 0x5EED
    plan.update(seeds, signs, torch.from_numpy(r).cuda(), W.alpha, sigma=sigma, flags=sr_flags,
                round_seed=round_seed)
    torch.cuda.synchronize()
    upd_sr = _gather(views, idx_dev)
    plan.close()
    del flat, views
    torch.cuda.empty_cache()

    reps = {"perturb": [], "swap": [], "restore": [], "update": [], "update_sr": []}
    for t, el_i in enumerate(idx):
        el = el_i.astype(np.uint64)
        exp = oracle.perturb(theta0[t], seed, t, sign, sigma, elems=el)
        reps["perturb"].append(report(pert[t], exp, theta0[t], perturb_delta(seed, t, sign, sigma, el)))
        exp = oracle.swap(pert[t], t, seed, sign, sigma, seed_b, sign_b, sigma, elems=el)
        dsw = perturb_delta(seed, t, -sign, sigma, el) + perturb_delta(seed_b, t, sign_b, sigma, el) \
            if seed != seed_b else perturb_delta(seed, t, sign_b - sign, sigma, el)
        reps["swap"].append(report(swp[t], exp, pert[t], dsw))
        exp = oracle.restore(swp[t], seed_b, t, sign_b, sigma, elems=el)
        reps["restore"].append(report(rest[t], exp, swp[t], perturb_delta(seed_b, t, -sign_b, sigma, el)))
        exp, st = oracle.update(rest[t], t, seeds, signs, r, W.alpha, sigma, elems=el)
        reps["update"].append(report(upd[t], exp, rest[t],
                                     update_delta(t, seeds, signs, r, W.alpha, sigma, 0, el)))
        exp, st = oracle.update(upd[t], t, seeds, signs, r, W.alpha, sigma, flags=sr_flags,
                                elems=el, round_seed=round_seed)
        reps["update_sr"].append(report(upd_sr[t], exp, upd[t],
                                        update_delta(t, seeds, signs, r, W.alpha, sigma, 0, el)))
    for k, rs in reps.items():
        n = sum(x["n"] for x in rs)
        agg = {
            "n": n,
            "exact": sum(x["exact"] * x["n"] for x in rs) / n,
            "le1": sum(x["le1"] * x["n"] for x in rs) / n,
            "max_ulp": max(x["max_ulp"] for x in rs),
            "plain_max_ulp": max(x["plain_max_ulp"] for x in rs),
            "n_gt1": sum(x["n_gt1"] for x in rs),
        }
        print(W.name, k, agg)
        assert_parity(agg, f"{W.name} {k}")


@pytest.mark.parametrize("name", ["dense-0.5b", "dense-4b", "dense-27b", "dense-27b-77l"])
def test_full_size_sampled_parity(name):
    _run(wl.WORKLOADS[name])


def test_large_population_sweep_n256_on_4b_set():
    _run(wl.sweep_workload(256), samples_per_tensor=64)


def test_single_tensor_beyond_2_34_elements():
    """One bf16 tensor of 2^34 + 4099 elements (32 GiB): past element 2^34 the
    quad index needs its high counter word and the draw group index passes
    2^31; elements on both sides of that boundary, of the last full tile and
    of the ragged tail are checked against the oracle after perturb, swap,
    restore and both update roundings, together with 20 000 random elements
    and both sides of the tensor's tile transitions."""
    n = (1 << 34) + 4099
    t = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    t.normal_(0.0, 0.02, generator=g)
    plan = esopt.Plan([t], tensor_ids=[77])
    b = 1 << 34
    edges, n_full, n_tail = _tile_edges(t)
    assert n_full > 0 and n_tail > 0
    # enough random samples for the bar's fractions to mean something
    # (>= 99.9 % bit-exact over 20 000 elements)
    idx = np.unique(np.concatenate([
        np.arange(0, 16), np.arange(b - 24, b + 24), np.arange(n - 4099 - 8, n - 4099 + 8),
        np.arange(n - 24, n), np.array(edges, dtype=np.int64),
        np.random.default_rng(1).integers(0, n, 20000)]).astype(np.int64))
    idx_dev = torch.from_numpy(idx).cuda()
    el = idx.astype(np.uint64)

    def gather():
        torch.cuda.synchronize()
        return to_host(t.index_select(0, idx_dev))
    x0 = gather()
    plan.perturb(11, -1, 1e-3)
    x1 = gather()
    plan.swap(11, -1, 12, 1, 1e-3)
    x2 = gather()
    plan.restore(12, 1, 1e-3)
    x3 = gather()
    r = np.array([0.2, 0.7, 0.4], np.float32)
    plan.update([3, 4, 5], [1, 1, 1], torch.from_numpy(r).cuda(), 5e-4)
    x4 = gather()
    plan.update([3, 4, 5], [1, 1, 1], torch.from_numpy(r).cuda(), 5e-4,
                flags=esopt.ES_UPDATE_STOCHASTIC_ROUND, round_seed=(1 << 63) + 9)
    x5 = gather()
    plan.close()
    del t
    torch.cuda.empty_cache()
    checks = [
        ("perturb", x1, oracle.perturb(x0, 11, 77, -1, 1e-3, elems=el), x0,
         perturb_delta(11, 77, -1, 1e-3, el)),
        ("swap", x2, oracle.swap(x1, 77, 11, -1, 1e-3, 12, 1, 1e-3, elems=el), x1,
         perturb_delta(11, 77, 1, 1e-3, el) + perturb_delta(12, 77, 1, 1e-3, el)),
        ("restore", x3, oracle.restore(x2, 12, 77, 1, 1e-3, elems=el), x2,
         perturb_delta(12, 77, -1, 1e-3, el)),
        ("update", x4, oracle.update(x3, 77, [3, 4, 5], [1, 1, 1], r, 5e-4, 1e-3, elems=el)[0], x3,
         update_delta(77, [3, 4, 5], [1, 1, 1], r, 5e-4, 1e-3, 0, el)),
        ("update_sr", x5, oracle.update(x4, 77, [3, 4, 5], [1, 1, 1], r, 5e-4, 1e-3, elems=el,
                                        flags=esopt.ES_UPDATE_STOCHASTIC_ROUND,
                                        round_seed=(1 << 63) + 9)[0], x4,
         update_delta(77, [3, 4, 5], [1, 1, 1], r, 5e-4, 1e-3, 0, el)),
    ]
    for name, got, exp, base, delta in checks:
        rep = report(got, exp, base, delta)
        print("2^34+", name, rep)
        assert_parity(rep, f"2^34+ {name}")
        assert rep["max_ulp"] <= 1.0, (name, rep)
    assert np.mean(x1 != x0) > 0.5
