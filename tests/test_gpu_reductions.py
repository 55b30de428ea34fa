"""The reductions around the sample (VEGAS histograms and grids, statistics,
unweighting, observable histograms) at the sizes where their splits of the
work change: bin counts around a wave, tile counts around the one-pass limit,
runs and remainders.  References: the oracle, or a plain numpy sum."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t

    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


@pytest.mark.parametrize("nb", [1, 2, 63, 64, 65, 128])
@pytest.mark.parametrize("n", [1, 63, 257, 17 * 256 * 4 + 5])
def test_vegas_accumulation_and_refinement(torch, nb, n):
    """The fused accumulation (one wave, partial waves, more tiles than the
    reduction has waves) and the refinement against the oracle's histogram of
    the sample's own weights and its refinement of it, and twice with the same
    bits.  Sums of n terms in another order: n times the unit roundoff of
    relative error, below 1e-11 here; the edges are sums of the damped shares,
    whose derivatives are of order one."""
    from paper_2602_06895_amd import SAMPLE_ACCUMULATE_VEGAS, Context

    desc = dict(W.c3_ttbar6(), vegas_bins=nb)
    grids = []
    for _ in range(2):
        ctx = Context(desc)
        out = ctx.sample([n], seed=5, stream_id=2, counter_offset=77, flags=SAMPLE_ACCUMULATE_VEGAS)
        ctx.vegas_update(0.5)
        grids.append(ctx.get_grid(0))
        w = out["w"].cpu().numpy()
        before = np.tile(np.arange(nb + 1) / nb, (ctx.dims[0], 1))
        ctx.close()
    assert np.array_equal(grids[0], grids[1])
    y = W.philox_uniforms(5, 2, 77, n, before.shape[0])
    want = oracle.vegas_refine(before, oracle.vegas_histogram(y, w, nb), 0.5)
    assert np.abs(grids[0] - want).max() <= 1e-10


@pytest.mark.parametrize("case", ["pp4j", "ttbar6", "chili", "dec3"])
@pytest.mark.parametrize("mixed", [False, True])
def test_sample_repeats_its_bits(torch, case, mixed):
    """The same call gives the same bits whatever ran in between (other
    contents of registers and LDS), with and without accumulation."""
    from paper_2602_06895_amd import FP64, MIXED, Context

    desc = W.c3_ttbar6() if case in ("ttbar6", "dec3") else W.c2_pp4j()
    if case == "chili":
        desc["channels"] = desc["channels"] + [{"chili": True}]
    if case == "dec3":
        desc["channels"] = [{"s": {"d": [{"d": [1, 2, 3], "m": 173.0, "w": 1.5, "order": 1},
                                         {"d": [4, 5, 6], "m": 173.0, "w": 1.5, "order": 2}]}}]
    ctx = Context(desc, precision=MIXED if mixed else FP64)
    counts = np.full(ctx.n_channels, 20011)
    for flags in (0, 1):
        ref = None
        for _ in range(3):
            torch.randn(1 << 22, device="cuda").sin_()
            out = ctx.sample(counts, seed=11, stream_id=4, counter_offset=123, flags=flags)
            bits = [out[k].view(torch.int64) for k in ("w", "p", "x1x2")]
            ref = ref or bits
            assert all(torch.equal(a, b) for a, b in zip(bits, ref))
    ctx.close()


@pytest.mark.parametrize("tiles", [1, 2047, 2048, 2049, 64 * 40, 64 * 40 + 1])
def test_statistics_of_many_tiles(torch, tiles):
    """One pass up to 2048 tiles of a channel, two beyond (full and ragged
    runs); beside a channel of one tile.  Relative error of a sum of n
    non-negative terms: at most n times the unit roundoff."""
    from paper_2602_06895_amd import Context

    desc = {"processes": [W.c1_ee_mumu(), W.c1_ee_mumu()]}
    ctx = Context(desc)
    counts = [256 * (tiles - 1) + 3, 100]
    out = ctx.sample(counts, seed=9, stream_id=1, counter_offset=5)
    st = ctx.stats()
    ctx.sample(counts, seed=9, stream_id=1, counter_offset=5)
    twice = ctx.stats()
    w = out["w"].cpu().numpy()
    off = 0
    for c, n in enumerate(counts):
        v = w[off:off + n]
        off += n
        tol = n * 2.0 ** -52
        for k, want in ((0, v.sum()), (1, (v * v).sum())):
            assert abs(st[c, k] - want) <= tol * want
            assert abs(twice[c, k] - 2.0 * want) <= 2.0 * tol * want
        assert st[c, 2] == n and st[c, 3] == (v == 0).sum() and st[c, 4] == v.max()
        assert twice[c, 2] == 2 * n and twice[c, 4] == v.max()
    ctx.close()


@pytest.mark.parametrize("kind", ["spread", "equal", "one", "ties"])
@pytest.mark.parametrize("n", [1, 2, 511, 4097, 512 * 512 + 1, 700_001])
def test_unweighting_efficiency_search(torch, kind, n):
    """The threshold against its definition on the sorted weights, the same
    bits on a second call.  The excess is linear in W between two weights, so
    W carries the relative error of the sums over the weights above it divided
    by their share of the total (1e-3): n times the unit roundoff times 1e3."""
    from paper_2602_06895_amd import Context

    rng = np.random.default_rng(n)
    w = {"spread": lambda: np.exp(rng.normal(0.0, 3.0, n)) * (rng.random(n) < 0.7),
         "equal": lambda: np.full(n, 0.37),
         "one": lambda: np.where(np.arange(n) == n // 2, 2.5, 0.0),
         "ties": lambda: rng.choice([1.0, 1.0 + 2.0 ** -52, 7.0, 1e-300], n)}[kind]()
    w[0] = max(w[0], 1e-3)
    ctx = Context(W.c1_ee_mumu())
    t = torch.from_numpy(w).cuda()
    got = [ctx.unweight_eff(t) for _ in range(2)]
    assert got[0] == got[1]
    eff, w_max = oracle.unweighting_efficiency(w)
    tol = 1e-12 + n * 2.0 ** -52 * 1e3
    assert abs(got[0][1] - w_max) <= tol * w_max and abs(got[0][0] - eff) <= tol * eff
    ctx.close()


@pytest.mark.parametrize("bins", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 4096])
@pytest.mark.parametrize("n", [0, 1, 63, 2049, 2048 * 2048 + 77])
def test_histogram_shapes(torch, bins, n):
    """One and four waves per workgroup, one, two and four histograms a wave, one bin, more bins than events, all
    events in one bin, values on the ends of the range; the same bits on a
    second call.  Sums of non-negative terms: n times the unit roundoff."""
    from paper_2602_06895_amd import Context

    rng = np.random.default_rng(n + bins)
    x = rng.normal(0.4, 0.3, n)
    w = np.exp(rng.normal(0.0, 1.0, n)) * (rng.random(n) < 0.6)
    if n > 8:
        x[:4] = [0.0, 1.0, np.nan, -0.0]
        x[n // 2:n // 2 + n // 4] = 0.5
        w[:4] = 1.0
    ctx = Context(W.c1_ee_mumu())
    tx, tw = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    a, b = (ctx.histogram(tx, tw, bins, 0.0, 1.0).cpu().numpy() for _ in range(2))
    assert np.array_equal(a, b)
    want = oracle.histogram(x, w, bins, 0.0, 1.0)
    assert np.all(np.abs(a - want) <= max(n, 1) * 2.0 ** -52 * want)
    ctx.close()


@pytest.mark.parametrize("nf", range(2, 9))
def test_observables_of_every_particle_count(torch, nf):
    """Every kind on full and partial sets, at every number of final-state
    particles, against the oracle.  Both sum the same doubles in the same order
    and differ by the rounding of a few library functions (1e-13 relative);
    the mass, whose E^2 - p^2 cancels, by u E^2 / M."""
    from paper_2602_06895_amd import (OBS_DR_HARDEST, OBS_E, OBS_ETA, OBS_M, OBS_PHI, OBS_PT, OBS_PT_RANK, Context)

    rng = np.random.default_rng(nf)
    n = 1003
    p = rng.normal(0.0, 50.0, (4, nf + 2, n))
    p[0] = np.sqrt((p[1:] ** 2).sum(0))
    p[1:, 3, :7] = p[1:, 2, :7]  # equal transverse momenta
    every, some = list(range(nf)), [0, nf - 1]
    spec = [(OBS_M, every, 0), (OBS_PT_RANK, every, nf - 1), (OBS_DR_HARDEST, every, 0), (OBS_ETA, [nf - 1], 0),
            (OBS_PHI, some, 0), (OBS_PT, every, 0), (OBS_E, some, 0), (OBS_PT_RANK, some, 1)]
    ctx = Context(W.volume_process(nf) if nf > 2 else W.c1_ee_mumu())
    got = ctx.observables(0, torch.from_numpy(p).cuda(), spec).cpu().numpy()
    want = oracle.observables(p, spec)
    scale = np.abs(want) + 1e-3  # angles and separations near zero: absolute
    scale[0] = want[0] + p[0, 2:].sum(0) ** 2 / np.maximum(want[0], 1e-3) * 1e-2
    assert np.all(np.abs(got - want) <= 1e-12 * scale)
    # a list that needs no energies and one that needs nothing but a sum of them
    for part in ([spec[2]], [spec[6]], [spec[4], spec[1]]):
        assert np.array_equal(ctx.observables(0, torch.from_numpy(p).cuda(), part).cpu().numpy(),
                              got[[spec.index(s) for s in part]])
    ctx.close()


@pytest.mark.parametrize("n", [1024, 1024 * 1024, 1024 * 1024 + 1, 1024 * 2049 + 5])
def test_unweighting_of_many_blocks(torch, n):
    """Runs of one, two and three blocks per thread of the offset scan: kept
    indices, unit weights and count equal to the oracle's."""
    from paper_2602_06895_amd import Context

    rng = np.random.default_rng(n)
    w = np.exp(rng.normal(0.0, 1.5, n)) * (rng.random(n) < 0.4)
    ctx = Context(W.c1_ee_mumu())
    out = ctx.unweight(torch.from_numpy(w).cuda(), 6.0, seed=3, stream_id=8, counter_offset=19)
    ref = oracle.unweight(w, 6.0, W.philox_uniforms(3, 8, 19, n, 1)[0])
    k = int(out["count"])
    assert k == len(ref["keep"])
    assert np.array_equal(out["keep"][:k].cpu().numpy(), ref["keep"])
    assert np.array_equal(out["uw"][:k].cpu().numpy(), ref["uw"])
    ctx.close()


@pytest.mark.parametrize("n_chan", [1, 2, 63, 64])
@pytest.mark.parametrize("counts", ["ragged", "full", "none", "over", "negative", "huge"])
def test_call_table_of_device_counts(torch, n_chan, counts):
    """The call table that one wave makes of device counts: the host call's
    events and statistics, the counter moved on by their number; refused counts
    (negative, over the capacity, sums beyond 64 bits) sample nothing.  Exact."""
    from paper_2602_06895_amd import SAMPLE_ADVANCE_COUNTER, Context

    cap = 20000
    desc = W.c1_ee_mumu()
    ctx = Context(dict(desc, channels=desc["channels"][:1] * n_chan))
    k = np.array([(257 * c) % 300 + (c % 3 == 0) for c in range(n_chan)], dtype=np.int64)
    if counts == "full":
        k[-1] += cap - k.sum()
    elif counts == "none":
        k[:] = 0
    elif counts == "over":
        k[-1] += cap - k.sum() + 1
    elif counts == "negative":
        k[n_chan // 2] = -1
    elif counts == "huge":
        k[:] = 2 ** 63 - 1
    buf = ctx.sample_buffers(cap)
    buf["w"].fill_(-7.0)
    off = torch.tensor([777], dtype=torch.int64, device="cuda")
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    ctx.sample_device(torch.from_numpy(k).cuda(), 9, 4, off, buf, status, flags=SAMPLE_ADVANCE_COUNTER)
    got = ctx.stats()
    refused = counts in ("over", "negative", "huge")
    n = 0 if refused else int(k.sum())
    assert int(status.cpu()[0]) == int(refused) and int(off.cpu()[0]) == 777 + n
    assert bool((buf["w"][n:] == -7.0).all())
    ctx.reset_stats()
    assert not ctx.stats().any()
    if n:
        ref = ctx.sample(k, seed=9, stream_id=4, counter_offset=777)
        assert np.array_equal(got, ctx.stats())
        assert torch.equal(buf["w"][:n], ref["w"]) and torch.equal(buf["chan"][:n], ref["chan"])
    else:
        assert not got.any()
    ctx.close()


@pytest.mark.parametrize("n", [1, 1000, 2049 * 256])
@pytest.mark.parametrize("desc", [W.c3_ttbar6, W.c2_pp4j])
def test_adaptation_is_its_steps(torch, n, desc):
    """msx_vegas_adapt against its steps called one by one, with old statistics
    in the context: the same statistics (one pass and two) and grids, exactly."""
    from paper_2602_06895_amd import SAMPLE_ACCUMULATE_VEGAS, Context, adapt_vegas

    a, b = Context(desc()), Context(desc())
    a.sample([5] * a.n_channels, seed=1, stream_id=1, counter_offset=0)
    got = adapt_vegas(a, n, 2, 0.5, 3, 2, 11)
    for it in range(2):
        b.reset_stats()
        b.sample([n] * b.n_channels, seed=3, stream_id=2, counter_offset=11 + it * n * b.n_channels,
                 flags=SAMPLE_ACCUMULATE_VEGAS)
        want = b.stats()
        b.vegas_update(0.5)
    assert np.array_equal(got, want) and not a.stats().any()
    for c in range(a.n_channels):
        assert np.array_equal(a.get_grid(c), b.get_grid(c))
    a.close()
    b.close()


def _nodes(torch, hip, call):
    """The number of nodes of the graph that `call` is captured into (hip:
    a library that is linked with the runtime)."""
    import ctypes as C

    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = C.c_size_t(0)
    assert hip.hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("flags", [0, 1, 2])
def test_device_count_sample_launches(torch, flags):
    """A device-count sample takes the same launches (call table, sample,
    statistics) whatever its buffers could hold."""
    from paper_2602_06895_amd import SAMPLE_ACCUMULATE_VEGAS, SAMPLE_ADVANCE_COUNTER, Context

    ctx = Context({"processes": [W.c1_ee_mumu(), W.c1_ee_mumu()]})
    fl = (0, SAMPLE_ACCUMULATE_VEGAS, SAMPLE_ADVANCE_COUNTER)[flags]
    counts = torch.tensor([700, 300], dtype=torch.int64, device="cuda")
    off = torch.zeros(1, dtype=torch.int64, device="cuda")
    nodes = []
    for cap in (1 << 20, 4000):
        buf = ctx.sample_buffers(cap)
        ctx.sample_device(counts, 3, 1, off, buf, flags=fl)
        torch.cuda.synchronize()
        nodes.append(_nodes(torch, ctx.L, lambda: ctx.sample_device(counts, 3, 1, off, buf, flags=fl)))
    assert nodes == [3, 3]
    ctx.close()


@pytest.mark.parametrize("vegas", [False, True])
def test_statistics_of_device_counts(torch, vegas):
    """The statistics of graph replays with many and few tiles in turn (slices and
    one step, ragged slices, no events), with eager calls in between: those of
    the host call of the same counts, exactly."""
    from paper_2602_06895_amd import SAMPLE_ACCUMULATE_VEGAS, Context

    a, b = (Context({"processes": [W.c1_ee_mumu()] * 3}) for _ in range(2))
    cap, fl = 256 * 9000, SAMPLE_ACCUMULATE_VEGAS if vegas else 0
    buf = a.sample_buffers(cap)
    counts = torch.zeros(3, dtype=torch.int64, device="cuda")
    off = torch.full((1,), 12, dtype=torch.int64, device="cuda")
    g = a.sample_graph(counts, 9, 1, off, buf, flags=fl)
    for k in ([256 * 2049, 5, 256 * 4000 + 1], [10, 256 * 2048, 0], [0, 0, 0], [256 * 2600 + 7, 256 * 3001, 256 * 2111],
              [1, 0, 256 * 8000]):
        counts.copy_(torch.tensor(k))
        a.reset_stats()
        b.reset_stats()
        g.launch()
        got = a.stats()
        if sum(k):
            b.sample(k, seed=9, stream_id=1, counter_offset=12, flags=fl)
        want = b.stats()
        assert np.array_equal(got, want) and list(got[:, 2]) == k
    g.close()
    a.close()
    b.close()


@pytest.mark.parametrize("bins", [1023, 1024, 1025, 2048])
@pytest.mark.parametrize("n", [1, 65, 2049, 300_007])
def test_histogram_with_helping_waves(torch, bins, n):
    """Around the number of bins from which three waves of a workgroup only clear
    and write out: as for the other shapes."""
    test_histogram_shapes(torch, bins, n)


@pytest.mark.parametrize("nf", range(2, 9))
def test_observables_of_short_and_long_lists(torch, nf):
    """Lists without ordered kinds that read as many particles as there are, one
    fewer and one more, which is where they change kernels: the bits of the
    same observables beside a rank, and the oracle's values within the bound of
    the test of all kinds."""
    from paper_2602_06895_amd import OBS_E, OBS_ETA, OBS_M, OBS_PHI, OBS_PT, OBS_PT_RANK, Context

    rng = np.random.default_rng(50 + nf)
    n = 777
    p = rng.normal(0.0, 50.0, (4, nf + 2, n))
    p[0] = np.sqrt((p[1:] ** 2).sum(0))
    dev = torch.from_numpy(p).cuda()
    every = list(range(nf))
    ctx = Context(W.volume_process(nf) if nf > 2 else W.c1_ee_mumu())
    lists = [[(k, every, 0)] for k in (OBS_E, OBS_PT, OBS_ETA, OBS_PHI, OBS_M)]
    lists += [[(OBS_M, every, 0), (OBS_PT, [nf - 1], 0)], [(OBS_ETA, every[1:], 0)],
              [(OBS_PT, [i], 0) for i in every], [(OBS_M, every[:2], 0), (OBS_PHI, [0], 0), (OBS_E, every[1:], 0)]]
    for spec in lists:
        got = ctx.observables(0, dev, spec).cpu().numpy()
        beside = ctx.observables(0, dev, spec[:7] + [(OBS_PT_RANK, every, 0)]).cpu().numpy()[:len(spec)]
        assert np.array_equal(got[:7], beside[:7])
        want = oracle.observables(p, spec)
        scale = np.abs(want) + 1e-3
        for j, (kind, s, _) in enumerate(spec):
            if kind == OBS_M:
                scale[j] += p[0, [2 + i for i in s]].sum(0) ** 2 / np.maximum(want[j], 1e-3) * 1e-2
        assert np.all(np.abs(got - want) <= 1e-12 * scale)
    ctx.close()


def _large(case):
    """Processes whose class kernels keep more than 256 registers."""
    ttbar = W.c3_ttbar6()
    three = {"s": {"d": [{"d": [1, 2, 3], "m": 173.0, "w": 1.5, "order": 1},
                         {"d": [4, 5, 6], "m": 173.0, "w": 1.5, "order": 2}]}}
    if case == "chili6":
        return W.chili_process(6, 13000.0, pt_min=20.0, pdf=[-1.2, 3.0])
    if case == "chili8":
        return W.chili_process(8, 13000.0, pt_min=20.0)
    if case == "vol8":
        return W.volume_process(8)
    if case == "ttbar6+chili":
        return dict(ttbar, channels=ttbar["channels"] + [{"chili": True}])
    if case == "ttbar6+dec3":
        return dict(ttbar, channels=ttbar["channels"] + [three])
    return dict(ttbar, channels=ttbar["channels"] + [three, {"chili": True}])


@pytest.mark.parametrize("case", ["chili6", "chili8", "vol8", "ttbar6+chili", "ttbar6+dec3", "all"])
@pytest.mark.parametrize("mixed", [False, True])
def test_sample_of_large_kernels_repeats_its_bits(torch, case, mixed):
    """As above, for the kernels with more than 256 registers; the map kernel of
    the last channel too."""
    from paper_2602_06895_amd import FP64, MIXED, Context

    ctx = Context(_large(case), precision=MIXED if mixed else FP64)
    counts = np.full(ctx.n_channels, 20011)
    c = ctx.n_channels - 1
    y = ctx.uniform(3, 1, 5, 20011, ctx.dims[c])
    for flags in (0, 1):
        ref = None
        for _ in range(3):
            torch.randn(1 << 22, device="cuda").sin_()
            out = ctx.sample(counts, seed=11, stream_id=4, counter_offset=123, flags=flags)
            m = ctx.map(c, y, weight=True)
            bits = [t.view(torch.int64).clone() for t in (out["w"], out["p"], m["p"], m["w"])]
            ref = ref or bits
            assert all(torch.equal(a, b) for a, b in zip(bits, ref))
    ctx.close()
