"""daso_fused_sync_step_noalloc (statistics scratch in the library's fixed device
array, no allocation) against daso_fused_sync_step on the same inputs: every
output bit for bit, on two calls in a row, the second one smaller, so that the
second call runs over partials the first left in the shared array."""
import numpy as np
import pytest
import torch

import paper_2104_05588_amd as daso
from oracle import daso_oracle as O
from workloads import generate as Gen
from workloads import recipes as R

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    daso.load()
    yield
    torch.cuda.synchronize()


def _random_case(seed, n, g, P, nb):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal(n) * 0.02).astype(F32)
    host = {"params": x, "momentum": (rng.standard_normal(n) * 1e-3).astype(F32),
            "grads": [(rng.standard_normal(n) * 1e-3).astype(F32) for _ in range(g)],
            "stale": [(torch.from_numpy(x + (rng.standard_normal(n) * 1e-4).astype(F32))
                       .to(torch.bfloat16).view(torch.int16)) for _ in range(P)]}
    cuts = sorted(set(rng.integers(1, n, nb - 1).tolist()))
    edges = [0] + cuts + [n]
    bks = [(edges[i], edges[i + 1] - edges[i], int(rng.choice([0, 1, 2, 4, 8]))) for i in range(len(edges) - 1)]
    bks = [bks[i] for i in rng.permutation(len(bks))]
    dev = {"params": torch.from_numpy(host["params"]).cuda(), "momentum": torch.from_numpy(host["momentum"]).cuda(),
           "grads": [torch.from_numpy(a).cuda() for a in host["grads"]],
           "stale": [t.cuda() for t in host["stale"]]}
    return dev, bks


def _workload_case(name):
    w = R.workload(name)
    return Gen.device_inputs(w), [(b.start, b.numel, b.S) for b in w.buckets]


def _run(inp, bks, noalloc):
    """One fused step on copies of the inputs; returns the outputs on the host."""
    n = inp["params"].numel()
    x, m = inp["params"].clone(), inp["momentum"].clone()
    wire = torch.empty(n, dtype=torch.int16, device="cuda")
    stats = daso.new_stats(len(bks))
    daso.fused_sync_step(inp["grads"], x, m, inp["stale"], bks, 0.1, 0.9, 0.0, wire, None, stats,
                         noalloc=noalloc)
    torch.cuda.synchronize()
    return {"params": x.cpu().numpy().view(np.uint32), "momentum": m.cpu().numpy().view(np.uint32),
            "wire": wire.cpu().numpy().view(np.uint16), "stats": stats.cpu().numpy().view(np.uint64)}


def _same(a, b, what):
    for k in ("params", "momentum", "wire", "stats"):
        diff = np.count_nonzero(a[k] != b[k])
        assert diff == 0, f"{what}: {k} differs in {diff} of {a[k].size} entries"


@pytest.mark.parametrize("first,second", [
    ("resnet50", "tiny"),                                  # full workload shapes, the bench's call first
    ((1, 1_000_003, 4, 8, 5), (2, 70_001, 3, 5, 3)),       # node shape, then a bounded instance
    ((3, 600_001, 8, 32, 7), (4, 4097, 9, 40, 2)),         # 1024-element tiles, then the run-time-count path
])
def test_noalloc_matches_fused_step_on_two_calls(first, second):
    cases = []
    for spec in (first, second):
        print(f"\n[case] noalloc vs fused: {spec}", flush=True)
        inp, bks = _workload_case(spec) if isinstance(spec, str) else _random_case(*spec)
        n = inp["params"].numel()
        cases.append((inp, bks, n))
    assert cases[1][2] < cases[0][2]
    # both calls of the fixed-scratch entry point back to back, then the reference calls
    got = [_run(inp, bks, noalloc=True) for inp, bks, _ in cases]
    for (inp, bks, n), g in zip(cases, got):
        want = _run(inp, bks, noalloc=False)
        _same(g, want, f"n={n} buckets={len(bks)}")


def test_noalloc_without_statistics_and_on_a_side_stream():
    inp, bks = _random_case(5, 300_007, 4, 4, 4)
    n = inp["params"].numel()
    want = _run(inp, bks, noalloc=False)
    x, m = inp["params"].clone(), inp["momentum"].clone()
    wire = torch.empty(n, dtype=torch.int16, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        daso.fused_sync_step(inp["grads"], x, m, inp["stale"], bks, 0.1, 0.9, 0.0, wire, None, None,
                             noalloc=True)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy().view(np.uint32), want["params"])
    assert np.array_equal(m.cpu().numpy().view(np.uint32), want["momentum"])
    assert np.array_equal(wire.cpu().numpy().view(np.uint16), want["wire"])


def test_noalloc_captures_in_a_graph_on_a_fresh_stream():
    """The fixed scratch needs no per-stream workspace, so the call can be
    captured on a stream that has never run a fused step (an eager call on
    another stream has looked up the scratch address on this device): every
    replay, with eager work and synchronisations between replays, gives the
    eager result bit for bit."""
    inp, bks = _random_case(6, 400_003, 4, 8, 3)
    n = inp["params"].numel()
    want = _run(inp, bks, noalloc=False)
    _same(_run(inp, bks, noalloc=True), want, "eager no-alloc call before the capture")
    x0, m0 = inp["params"], inp["momentum"]
    x, m = x0.clone(), m0.clone()
    wire = torch.empty(n, dtype=torch.int16, device="cuda")
    stats = daso.new_stats(len(bks))
    step = daso.FusedStep(inp["grads"], x, m, inp["stale"], bks, 0.1, 0.9, 0.0, wire=wire, stats=stats,
                          noalloc=True)
    fresh = torch.cuda.Stream()
    fresh.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=fresh):
        step()
    torch.cuda.synchronize()
    for rep in range(3):
        x.copy_(x0)
        m.copy_(m0)
        wire.fill_(0)
        stats.zero_()
        if rep == 1:   # other eager work on the device between replays
            _run(inp, bks, noalloc=True)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(x.cpu().numpy().view(np.uint32), want["params"]), rep
        assert np.array_equal(m.cpu().numpy().view(np.uint32), want["momentum"]), rep
        assert np.array_equal(wire.cpu().numpy().view(np.uint16), want["wire"]), rep
        assert np.array_equal(stats.cpu().numpy().view(np.uint64), want["stats"]), rep


def _device_case(seed, n, g, P):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(sigma):
        return torch.randn(n, generator=gen, device="cuda", dtype=torch.float32).mul_(sigma)
    x = normal(0.02)
    return {"params": x, "momentum": normal(1e-3), "grads": [normal(1e-3) for _ in range(g)],
            "stale": [(x + normal(1e-4)).to(torch.bfloat16).view(torch.int16) for _ in range(P)]}


def test_noalloc_with_more_buckets_than_its_array_holds():
    """170,000 buckets of one to three elements: their partials exceed the fixed array
    and what the allocated workspace shares, so each launch of 128 buckets has a
    statistics pass of its own, over the places that the one before used.  Both entry
    points against the oracle, taken once per staleness over the whole set."""
    starts = np.concatenate([[0], np.cumsum([1 + k % 3 for k in range(170_000)])])
    n = int(starts[-1])
    sizes, S = np.diff(starts), np.array([(1, 2, 4)[k % 5 % 3] for k in range(170_000)])
    bks = [(int(a), int(k), int(s)) for a, k, s in zip(starts, sizes, S)]
    print(f"\n[case] noalloc, {len(bks)} buckets, n={n}", flush=True)
    inp = _device_case(21, n, 4, 2)
    host = {k: [t.cpu().numpy() for t in v] if isinstance(v, list) else v.cpu().numpy() for k, v in inp.items()}
    stale = [t.view(np.uint16) for t in host["stale"]]
    gbar = O.local_avg(host["grads"])
    xl, m = O.sgd_momentum(host["params"], host["momentum"], gbar, 0.1, 0.9, 0.0)
    each = np.repeat(S, sizes)
    x = np.choose(np.searchsorted([1, 2, 4], each), [O.merge_eq1(xl, stale, s) for s in (1, 2, 4)])
    delta = x.astype(np.float64) - xl.astype(np.float64)
    sums = np.stack([np.add.reduceat(np.square(v), starts[:-1]) for v in (gbar.astype(np.float64), delta)], axis=1)
    for noalloc in (True, False):
        got = _run(inp, bks, noalloc=noalloc)
        assert np.array_equal(got["params"], x.view(np.uint32))
        assert np.array_equal(got["momentum"], m.view(np.uint32))
        assert np.array_equal(got["wire"], O.bf16_rne(x))
        assert not got["stats"][:, 2].any()
        # at most three squares each, added in another order
        np.testing.assert_allclose(got["stats"].view(np.float64)[:, :2], sums, rtol=2.0 ** -51, atol=0)


def test_noalloc_with_a_bucket_whose_partials_exceed_its_array():
    """A bucket of 740 million parameters between two others: the array holds the partials of
    715 million, so the bucket takes two launches whose statistics are added up.
    Every other output is the same, the statistics up to the order of their sums."""
    n = 740_000_003
    bks = [(0, 5_003, 1), (5_003, n - 12_000, 2), (n - 6_997, 6_997, 1)]
    print(f"\n[case] noalloc, a bucket of {n - 12_000}", flush=True)
    inp = _device_case(22, n, 1, 0)
    for nonfinite in (2, 0):
        inp["grads"][0][n // 2] = float("inf") if nonfinite else 1e-3    # in the first part
        inp["grads"][0][n - 7_100] = float("nan") if nonfinite else 1e-3  # in the second
        outs = []
        for noalloc in (True, False):
            x, m = inp["params"].clone(), inp["momentum"].clone()
            stats = daso.new_stats(len(bks))
            daso.fused_sync_step(inp["grads"], x, m, [], bks, 0.1, 0.9, stats=stats, noalloc=noalloc)
            torch.cuda.synchronize()
            outs.append((x, m, daso.decode_stats(stats)))
        for k in (0, 1):
            assert torch.equal(outs[0][k].view(torch.int32), outs[1][k].view(torch.int32))
        for b, (got, want) in enumerate(zip(outs[0][2], outs[1][2])):
            assert got[2] == want[2] == (nonfinite if b == 1 else 0)
            if b != 1:
                assert got == want
            elif not nonfinite:
                # 700,000 partials in trees of fewer than 800 additions one after the other: 800 * 2^-53
                assert 0 < want[0] and abs(got[0] - want[0]) <= 1e-13 * want[0]
                assert got[1] == want[1] == 0.0  # nothing merged
        del outs
