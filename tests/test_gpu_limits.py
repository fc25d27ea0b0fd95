"""Plans at the limits.  The maximum tensor count (ES_MAX_TENSORS = 2^20): views of 0 to
8 elements each, every one a tail tile of its own.  Perturb and update leave
the same bits as the same tensors planned in reverse order (the noise depends
only on each tensor's id and element index), sampled tensors match the
oracle, and the bytes between the views are untouched.  And a plan of more
elements than one launch of the update covers."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_17310_amd import esopt, workloads as wl
from parity import assert_parity, perturb_delta, report, to_device, to_host, update_delta

pytestmark = pytest.mark.gpu

MAX_TENSORS = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def test_plan_at_the_maximum_tensor_count():
    rng = np.random.default_rng(90)
    sizes = rng.integers(0, 9, MAX_TENSORS)
    starts = np.arange(MAX_TENSORS) * 10 + rng.integers(0, 2, MAX_TENSORS)   # some unaligned
    bits = wl.random_bf16_bits(MAX_TENSORS * 10 + 8, 91)
    ids = rng.permutation(1 << 24)[:MAX_TENSORS]
    r = torch.tensor([0.3, 0.8, 0.1, 0.6], device="cuda")
    outs, mid = [], None
    for order in (1, -1):
        buf = to_device(bits)
        views = [buf[s:s + n] for s, n in zip(starts, sizes)]
        with esopt.Plan(views[::order], tensor_ids=list(ids[::order])) as p:
            assert p.numel == int(sizes.sum())
            p.perturb(12, -1, 1e-3)
            if order == 1:
                torch.cuda.synchronize()
                mid = to_host(buf)
            p.update([1, 2, 2, 3], [1, 1, -1, 1], r, 5e-4)
        torch.cuda.synchronize()
        outs.append(to_host(buf))
        del views
    np.testing.assert_array_equal(outs[0], outs[1])
    gaps = np.ones(bits.size, bool)
    for s, n in zip(starts, sizes):
        gaps[s:s + n] = False
    np.testing.assert_array_equal(outs[0][gaps], bits[gaps])
    # sampled tensors, each pass against the oracle applied to the GPU's
    # state before it
    reps = {"perturb": ([], [], [], []), "update": ([], [], [], [])}
    rr = r.cpu().numpy()
    for k in rng.choice(MAX_TENSORS, 400, replace=False):
        s, n, t = int(starts[k]), int(sizes[k]), int(ids[k])
        if n == 0:
            continue
        el = np.arange(n, dtype=np.uint64)
        x0, x1, x2 = bits[s:s + n], mid[s:s + n], outs[0][s:s + n]
        for name, got, exp, base, d in (
                ("perturb", x1, oracle.perturb(x0, 12, t, -1, 1e-3, elems=el), x0,
                 perturb_delta(12, t, -1, 1e-3, el)),
                ("update", x2, oracle.update(x1, t, [1, 2, 2, 3], [1, 1, -1, 1], rr, 5e-4, 1e-3,
                                             elems=el)[0], x1,
                 update_delta(t, [1, 2, 2, 3], [1, 1, -1, 1], rr, 5e-4, 1e-3, 0, el))):
            for lst, v in zip(reps[name], (got, exp, base, d)):
                lst.append(v)
    for name, lists in reps.items():
        rep = report(*[np.concatenate(v) for v in lists])
        print("2^20 tensors, sampled:", name, rep)
        assert_parity(rep, name)


def test_quantized_plan_at_the_maximum_tensor_count():
    """The same for an int8 plan: 2^20 views of 0 to 40 codes sharing one
    scale, each a tail tile of its own (the table lookup per tile at its
    largest), order-independent codes, untouched gaps, sampled oracle parity
    of the perturbation."""
    from test_gpu_quant import _perturb_expect
    from parity import assert_qparity, qreport
    rng = np.random.default_rng(92)
    sizes = rng.integers(0, 41, MAX_TENSORS)
    starts = np.arange(MAX_TENSORS) * 48 + rng.integers(0, 3, MAX_TENSORS)
    codes = rng.integers(-127, 128, MAX_TENSORS * 48 + 8).astype(np.int8)
    ids = rng.permutation(1 << 24)[:MAX_TENSORS]
    scale = np.array([6e-4], np.float32)
    r = torch.tensor([0.3, 0.8, 0.1], device="cuda")
    outs, mid = [], None
    for order in (1, -1):
        buf = torch.from_numpy(codes).cuda()
        views = [buf[s:s + n] for s, n in zip(starts, sizes)]
        sdev = torch.from_numpy(scale).cuda()
        with esopt.QPlan(views[::order], [sdev] * MAX_TENSORS, [0] * MAX_TENSORS,
                         tensor_ids=list(ids[::order])) as p:
            assert p.numel == int(sizes.sum())
            p.perturb(13, 1, 1e-3)
            if order == 1:
                torch.cuda.synchronize()
                mid = buf.cpu().numpy()
            p.update([1, 2, 3], [1, -1, 1], r, 5e-4, round_seed=4)
        torch.cuda.synchronize()
        outs.append(buf.cpu().numpy())
        del views
    np.testing.assert_array_equal(outs[0], outs[1])
    gaps = np.ones(codes.size, bool)
    for s0, n in zip(starts, sizes):
        gaps[s0:s0 + n] = False
    np.testing.assert_array_equal(outs[0][gaps], codes[gaps])
    got, q_in, v, tol, ok = [], [], [], [], []
    for k in rng.choice(MAX_TENSORS, 400, replace=False):
        s0, n, t = int(starts[k]), int(sizes[k]), int(ids[k])
        if n == 0:
            continue
        d, o, tl = _perturb_expect(scale, 0, 13, t, 1, 1e-3, np.arange(n, dtype=np.uint64))
        for lst, x in zip((got, q_in, v, tol, ok), (mid[s0:s0 + n], codes[s0:s0 + n], d, tl, o)):
            lst.append(x)
    rep = qreport(*[np.concatenate(x) for x in (got, q_in, v, tol, ok)])
    print("2^20 int8 tensors, sampled perturb:", rep)
    assert_qparity(rep, "int8 perturb at 2^20 tensors")



def test_update_of_a_plan_beyond_one_launch():
    """2^36 elements and some (137 GB): an update's one-step workgroups would
    have 2^32 lanes there, more than a launch takes, so the pass is two launches.
    Elements around the start, the cut between them, a counter's high word and
    the end, each pass against the oracle."""
    n = (1 << 36) + 3 * 65536 + 4099
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 2 * n + (8 << 30):
        pytest.skip("not enough free device memory")
    t = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    first_launch = ((1 << 24) - 1) // 16 * 65536          # elements in its whole tiles
    marks = [0, 1 << 34, first_launch - 65536, first_launch, 1 << 36, n - 9000]
    at = np.unique(np.concatenate([np.arange(max(0, m - 4500), min(n, m + 9000), dtype=np.uint64)
                                   for m in marks]))
    runs = np.split(at, np.flatnonzero(np.diff(at) > 1) + 1)
    bits = wl.random_bf16_bits(at.size, 93)

    def spans():
        return [t[int(r[0]):int(r[-1]) + 1] for r in runs]
    done = 0
    for v in spans():
        v.copy_(to_device(bits[done:done + v.numel()]))
        done += v.numel()

    def host():
        torch.cuda.synchronize()
        return np.concatenate([to_host(v) for v in spans()])
    seeds, signs, rr = [1, 2, 1], [1, 1, -1], np.array([0.3, 0.8, 0.1], np.float32)
    r = torch.from_numpy(rr).cuda()
    with esopt.Plan([t], tensor_ids=[5]) as p:
        p.perturb(2, 1, 1e-3)
        x1 = host()
        assert_parity(report(x1, oracle.perturb(bits, 2, 5, 1, 1e-3, elems=at), bits,
                             perturb_delta(2, 5, 1, 1e-3, at)), "perturb beyond 2^36")
        p.restore(2, 1, 1e-3)
        x2 = host()
        assert_parity(report(x2, oracle.restore(x1, 2, 5, 1, 1e-3, elems=at), x1,
                             perturb_delta(2, 5, -1, 1e-3, at)), "restore beyond 2^36")
        p.update(seeds, signs, r, 5e-4)
        x3 = host()
    assert_parity(report(x3, oracle.update(x2, 5, seeds, signs, rr, 5e-4, 1e-3, elems=at)[0], x2,
                         update_delta(5, seeds, signs, rr, 5e-4, 1e-3, 0, at)),
                  "update beyond 2^36")
    # 256 elements in every 2^30 held zeros, which the passes left as noise
    far = torch.stack([t[k << 30:(k << 30) + 256] for k in range(1, 64)])
    del t
    torch.cuda.empty_cache()                            # the library allocates outside the cache
    assert int((far != 0).sum()) > 0.99 * far.numel()
