"""The step's split into pieces of 256 elements at the sizes where it can go
wrong: around a piece, a superblock of 2048 or 8192 elements and the 16-byte
vector, with buckets that begin and end inside a piece, several in one piece and
empty ones, for every kind of instance (exact, bounded and unbounded counts, with one,
four and eight wavefronts per workgroup, both exchange types); tables of more buckets than one
launch takes; and launches of small buckets alone.  Against the oracle, bit for bit (statistics: fp64 sums in another order,
1e-10)."""
import numpy as np
import pytest
import torch

import paper_2104_05588_amd as daso
from oracle import daso_oracle as O
from tests.test_gpu_parity import (F32, announce, check_f32, check_stats, check_u16, compare_fused, dev_bf16, dev_f32,
                                   host_f32, host_u16, random_inputs, run_fused)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    daso.load()
    yield
    torch.cuda.synchronize()


SIZES = [1, 255, 256, 257, 2047, 2048, 2051, 8190, 8192, 8197, 16_384, 24_579]


def edge_buckets(rng, n):
    """Buckets tiling [0, n) whose edges lie on, just before and just after the
    split's own, with a few of one to three elements and an empty one, in random order."""
    near = [e + d for e in range(0, n + 1, 256) for d in (-3, -1, 0, 1) if 0 < e + d < n]
    cuts = sorted(set(rng.choice(near, min(len(near), 12), replace=False).tolist())) if near else []
    if cuts:
        cuts = sorted(set(cuts + [c + 1 for c in cuts[:2] if c + 1 < n] + [c + 3 for c in cuts[:2] if c + 3 < n]))
    edges = [0] + cuts + [n]
    bks = [(a, b - a, int(rng.choice((0, 1, 2, 3, 8)))) for a, b in zip(edges[:-1], edges[1:])]
    bks.append((edges[len(edges) // 2], 0, 5))
    return [bks[i] for i in rng.permutation(len(bks))]


@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.parametrize("g,P,f32", [(4, 8, False), (8, 32, False), (4, 64, False), (3, 5, False), (6, 21, False),
                                     (9, 3, False), (2, 45, False), (4, 0, False), (8, 16, True), (5, 11, True),
                                     (4, 33, True)])
def test_pieces_at_their_edges(g, P, f32, stats):
    rng = np.random.default_rng(1000 * g + 10 * P + stats)
    for n in SIZES:
        bks = edge_buckets(rng, n)
        inp = random_inputs(rng, n, g, P)
        if f32:
            inp["stale"] = [O.bf16_widen(s) + F32(1e-6) for s in inp["stale"]]
        announce("pieces g=", g, "P=", P, "f32" if f32 else "bf16", "stats" if stats else "", "n=", n, "buckets",
                 len(bks))
        want = O.fused_sync_step(inp["grads"], inp["params"], inp["momentum"], inp["stale"], bks, 0.1, 0.9, 1e-4,
                                 exchange="f32" if f32 else "bf16")
        got = run_fused(inp, bks, wd=1e-4, gavg="alias", stats=stats, f32=f32)
        compare_fused(got, want, f"pieces g={g} P={P} n={n}", gavg=True, stats=stats)


@pytest.mark.parametrize("stats", [False, True])
@pytest.mark.parametrize("g,P,f32", [(8, 32, False), (4, 64, False), (4, 16, True), (8, 32, True), (9, 3, False),
                                     (2, 45, False), (4, 33, True)])
def test_last_pieces_of_whole_vectors(g, P, f32, stats):
    """Calls that end inside a piece at a multiple of 4, whose last vectors are read whole, with
    buckets that meet inside a vector and without, several of them in one piece, whose vectors
    unbounded counts then take in one pass; and at an odd element, read one by one."""
    rng = np.random.default_rng(3000 * g + 10 * P + stats)
    for n in (4, 252, 260, 1028, 8188, 8196, 30_000, 30_001):
        tables = [[(0, n, 2)], [(0, n - 4, 1), (n - 4, 4, 0)], [(n - 3, 3, 3), (0, n - 3, 1)]]
        if n >= 30_000:
            cuts = [0, 20_000, 20_004, 20_052, 20_052, 20_152, n]
            tables.append([(s, e - s, k % 4) for k, (s, e) in enumerate(zip(cuts, cuts[1:]))])
        for bks in tables:
            inp = random_inputs(rng, n, g, P)
            if f32:
                inp["stale"] = [O.bf16_widen(s) + F32(1e-6) for s in inp["stale"]]
            announce("last piece g=", g, "P=", P, "f32" if f32 else "bf16", "stats" if stats else "", "n=", n)
            want = O.fused_sync_step(inp["grads"], inp["params"], inp["momentum"], inp["stale"], bks, 0.1, 0.9, 1e-4,
                                     exchange="f32" if f32 else "bf16")
            got = run_fused(inp, bks, wd=1e-4, gavg="alias", stats=stats, f32=f32)
            compare_fused(got, want, f"last piece g={g} P={P} n={n}", gavg=True, stats=stats)
            want, wire = O.global_merge(inp["params"], inp["stale"], bks, pack=True, exchange="f32" if f32 else "bf16")
            xd = dev_f32(inp["params"])
            wd = torch.empty(n, dtype=torch.float32 if f32 else torch.int16, device="cuda")
            daso.global_merge(xd, [(dev_f32 if f32 else dev_bf16)(s) for s in inp["stale"]], bks, wd)
            torch.cuda.synchronize()
            check_f32(host_f32(xd), want, f"merge of P={P} n={n}")
            if f32:
                check_f32(host_f32(wd), wire, f"wire of P={P} n={n}")
            else:
                check_u16(host_u16(wd), wire, f"wire of P={P} n={n}")


@pytest.mark.parametrize("g,P,f32", [(8, 32, False), (4, 16, True)])
@pytest.mark.parametrize("n", [3 << 20, (3 << 20) + 1, (3 << 20) + 12_292])
def test_workgroups_of_eight_begin_beyond_a_short_call(g, P, f32, n):
    """The longest call in workgroups of four wavefronts, and calls in eights that end in a
    superblock's first vector and last workgroups, with buckets that meet inside a piece."""
    rng = np.random.default_rng(n + g)
    bks = [(0, 300, 2), (300, 1_500_003, 0), (1_500_303, n - 1_500_303, 1)]
    inp = random_inputs(rng, n, g, P)
    if f32:
        inp["stale"] = [O.bf16_widen(s) + F32(1e-6) for s in inp["stale"]]
    announce("eights g=", g, "P=", P, "f32" if f32 else "bf16", "n=", n)
    want = O.fused_sync_step(inp["grads"], inp["params"], inp["momentum"], inp["stale"], bks, 0.1, 0.9, 1e-4,
                             exchange="f32" if f32 else "bf16")
    got = run_fused(inp, bks, wd=1e-4, gavg="new", stats=True, f32=f32)
    compare_fused(got, want, f"eights g={g} P={P} n={n}", gavg=True, stats=True)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("P", [1, 2, 4, 5, 8, 12, 16, 20, 32, 40])
def test_mean_of_copies_at_its_edges(P, f32):
    """One staleness 0 for every bucket: the average of the copies, into parameters that
    are NaN before.  Without a wire, as blocking_average calls it, the instances that do not read the
    parameters (every exact, bounded and unbounded count); with one, the merge with S = 0."""
    rng = np.random.default_rng(70 + P)
    for n in SIZES:
        announce("mean P=", P, "f32" if f32 else "bf16", "n=", n)
        bks = [(s, k, 0) for s, k, _ in edge_buckets(rng, n)]
        st = random_inputs(rng, n, 1, P)["stale"]
        if f32:
            st = [O.bf16_widen(s) + F32(1e-6) for s in st]
        x = np.full(n, np.nan, F32)
        want, wire = O.global_merge(x, st, bks, pack=True, exchange="f32" if f32 else "bf16")
        sd = [(dev_f32 if f32 else dev_bf16)(s) for s in st]
        xd = dev_f32(x)
        daso.global_merge(xd, sd, bks)
        torch.cuda.synchronize()
        check_f32(host_f32(xd), want, f"mean P={P} n={n}")
        xd, wd = dev_f32(x), torch.empty(n, dtype=torch.float32 if f32 else torch.int16, device="cuda")
        daso.global_merge(xd, sd, bks, wd)
        torch.cuda.synchronize()
        check_f32(host_f32(xd), want, f"merge with S = 0, P={P} n={n}")
        if f32:
            check_f32(host_f32(wd), wire, f"wire of a merge with S = 0, P={P} n={n}")
        else:
            check_u16(host_u16(wd), wire, f"wire of a merge with S = 0, P={P} n={n}")


@pytest.mark.parametrize("nb,n", [(127, 300_001), (129, 300_001), (400, 90_001), (1100, 50_003)])
def test_statistics_of_more_buckets_than_a_launch(nb, n):
    """Several launches share one statistics pass; the no-alloc entry point gives the
    same bits."""
    rng = np.random.default_rng(nb)
    cuts = sorted(rng.choice(np.arange(1, n), nb - 1, replace=False).tolist())
    edges = [0] + cuts + [n]
    bks = [(a, b - a, int(rng.choice((1, 2, 4)))) for a, b in zip(edges[:-1], edges[1:])]
    bks = [bks[i] for i in rng.permutation(nb)]
    inp = random_inputs(rng, n, 4, 4)
    announce("statistics of", nb, "buckets, n=", n)
    want = O.fused_sync_step(inp["grads"], inp["params"], inp["momentum"], inp["stale"], bks, 0.1, 0.9)
    compare_fused(run_fused(inp, bks), want, f"{nb} buckets")
    bits = []
    for noalloc in (False, True):
        x, m, st = dev_f32(inp["params"]), dev_f32(inp["momentum"]), daso.new_stats(nb)
        daso.fused_sync_step([dev_f32(a) for a in inp["grads"]], x, m, [dev_bf16(s) for s in inp["stale"]], bks,
                             0.1, 0.9, stats=st, noalloc=noalloc)
        torch.cuda.synchronize()
        check_f32(host_f32(x), want["params"], f"{nb} buckets noalloc={noalloc}")
        check_stats(daso.decode_stats(st), want["stats"], f"{nb} buckets noalloc={noalloc}")
        bits.append(st.cpu().numpy().view(np.uint64))
    assert np.array_equal(bits[0], bits[1])


@pytest.mark.parametrize("g,P,S", [(3, 3, 1), (5, 7, 4), (7, 5, 3), (6, 1, 1)])
def test_division_of_tiny_zero_and_special_values(g, P, S):
    """Quotients by counts that are no power of two, of values from the smallest
    subnormal over the 2^-100 below which the plain division is taken to the
    largest, zeros of both signs, infinities and NaN: correctly rounded."""
    rng = np.random.default_rng(100 * g + P)
    n = 40_003
    announce("division g=", g, "P=", P, "S=", S)

    def values():
        v = (rng.standard_normal(n) * np.exp2(rng.uniform(-149, 127, n))).astype(F32)
        v[rng.integers(0, n, 200)] = rng.choice(
            np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 2.0 ** -149, -2.0 ** -126, 2.0 ** -100], F32), 200)
        v[:8192] = np.where(np.abs(v[:8192]) < 2.0 ** -90, F32(0.25), v[:8192])  # pieces without tiny values
        return v

    with np.errstate(all="ignore"):
        grads = [values()] + [np.zeros(n, F32) for _ in range(g - 1)]
        stale = [O.bf16_rne(values())] + [np.zeros(n, np.uint16) for _ in range(P - 1)]
        inp = {"params": np.zeros(n, F32), "momentum": np.zeros(n, F32), "grads": grads, "stale": stale}
        bks = [(0, n, S)]
        want = O.fused_sync_step(grads, inp["params"], inp["momentum"], stale, bks, 1e-30, 0.9)
        got = run_fused(inp, bks, lr=1e-30, gavg="new", stats=False)
        compare_fused(got, want, f"division g={g} P={P}", gavg=True, stats=False)


@pytest.mark.parametrize("g,P,f32", [(4, 8, False), (1, 0, False), (9, 40, False), (4, 3, True)])
@pytest.mark.parametrize("stats", [False, True])
def test_launches_of_small_buckets(g, P, f32, stats):
    """Launches whose buckets are all small take wavefronts of each bucket's own: buckets of no
    elements to the most (on average and alone) for each kind of instance and just beyond,
    in launches by themselves and beside others in one call, whose statistics pass must leave
    theirs as they are."""
    rng = np.random.default_rng(31 * g + P + stats)
    for sizes in ([1] * 300, list(range(0, 130)) * 2, [128, 0] * 65, [129, 1, 1, 1], [2, 1], [64] * 9, [65] * 9,
                  [2048, 0, 1] * 45, [2049, 1, 1], [4096, 1, 0] * 3, [4097, 1, 1], [6144, 3, 5], [6145, 1, 1, 255], [3072, 3072, 3073],
                  [40] * 128 + [15000, 7] + [3] * 126 + [257, 1] * 64, [30] * 127 + [9001] + [30] * 200,
                  [9000, 5, 700, 3, 9000, 4], [9000, 5, 700, 3, 9000, 1, 2]):
        bks, pos = [], 0
        for k in sizes:
            bks.append((pos, k, int(rng.choice((0, 1, 2, 3)))))
            pos += k
        inp = random_inputs(rng, pos, g, P)
        if f32:
            inp["stale"] = [O.bf16_widen(s) + F32(1e-6) for s in inp["stale"]]
        announce("small buckets g=", g, "P=", P, "f32" if f32 else "bf16", "stats" if stats else "", "buckets",
                 len(bks), "n=", pos)
        order = rng.permutation(len(bks))
        for table, gavg in ((bks, "alias"), ([bks[i] for i in order], "new")):
            want = O.fused_sync_step(inp["grads"], inp["params"], inp["momentum"], inp["stale"], table, 0.1, 0.9, 1e-4,
                                     exchange="f32" if f32 else "bf16")
            got = run_fused(inp, table, wd=1e-4, gavg=gavg, stats=stats, f32=f32)
            compare_fused(got, want, f"small buckets g={g} P={P} n={pos}", gavg=True, stats=stats)
        if not stats and not f32:
            want, wire = O.global_merge(inp["params"], inp["stale"], bks, pack=True)
            xd, wd = dev_f32(inp["params"]), torch.empty(pos, dtype=torch.int16, device="cuda")
            daso.global_merge(xd, [dev_bf16(s) for s in inp["stale"]], bks, wd)
            torch.cuda.synchronize()
            check_f32(host_f32(xd), want, f"merge of small buckets P={P} n={pos}")
            check_u16(host_u16(wd), wire, f"merge wire of small buckets P={P} n={pos}")


def test_captured_call_of_more_buckets_than_its_warm_up():
    """An eager call with one bucket warms the stream up; the captured one has 3000, whose
    partials and table exceed the workspace, so its launches take a statistics pass each.
    Every replay, with eager work between, gives the bits of an eager call with them."""
    n, size = 20_000_001, 6_667
    bks = [(s, min(size, n - s), 1 + s // size % 3) for s in range(0, n, size)]
    announce("captured", len(bks), "buckets after one, n=", n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x0 = torch.randn(n, generator=gen, device="cuda") * 0.02
    m0 = torch.randn(n, generator=gen, device="cuda") * 1e-3
    grads = [torch.randn(n, generator=gen, device="cuda") * 1e-3 for _ in range(2)]
    stale = [(x0 + 1e-4).to(torch.bfloat16) for _ in range(3)]
    x, m = x0.clone(), m0.clone()
    one, stats = daso.new_stats(1), daso.new_stats(len(bks))
    step = daso.FusedStep(grads, x, m, stale, bks, 0.1, 0.9, stats=stats)
    step()                                             # on another stream
    torch.cuda.synchronize()
    eager = (x.clone(), m.clone(), stats.clone())
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        daso.fused_sync_step(grads, x, m, stale, [(0, n, 1)], 0.1, 0.9, stats=one)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(3):
        x.copy_(x0)
        m.copy_(m0)
        stats.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(x.view(torch.int32), eager[0].view(torch.int32)), rep
        assert torch.equal(m.view(torch.int32), eager[1].view(torch.int32)), rep
        assert torch.equal(stats.view(torch.int64), eager[2].view(torch.int64)), rep
        with torch.cuda.stream(side):                  # other work in the same workspace
            daso.fused_sync_step(grads, x, m, stale, [(0, n, 1)], 0.1, 0.9, stats=one)
        torch.cuda.synchronize()
