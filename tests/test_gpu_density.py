"""The multichannel density where its channels are split into launches: more
channels of a class than a launch takes, scratch that holds fewer than a run, the
one-channel fallback, and captured calls beside eager ones that use the same
scratch.  The reference is the sum of alpha / J over the channels, one at a
time and in order, with J from msx_inverse_map: the same operations on the same
numbers, so the bits are equal."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t

    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


def _events(ctx, n, seed, chan=0):
    y = ctx.uniform(seed, 3, 0, n, ctx.dims[chan])
    out = ctx.map(chan, y)
    return out["p"], out["x1x2"]


def _one_by_one(torch, ctx, chans, p, x, alpha):
    g = torch.zeros(p.shape[2], dtype=torch.float64, device="cuda")
    for c, a in zip(chans, alpha):
        j = ctx.inverse_map(c, p, x)["jac"]
        g = g + torch.where(j > 0, torch.full_like(j, a) / j, torch.zeros_like(j))
    return g


@pytest.mark.parametrize("chans,n", [(list(range(8)), 3), (list(range(8)) * 2, 300), (list(range(8)) * 2 + [3], 1000),
                                     ([6] * 30 + [0, 6], 257), (list(range(8)), 3_300_001)])
def test_density_of_split_runs(torch, chans, n):
    """One run, 16, 17 and 32 channels of a class; at 3.3 million events the 2
    GiB hold seven of the eight channels."""
    from paper_2602_06895_amd import Context

    desc = W.c2_pp4j()
    desc["channels"] = [desc["channels"][c] for c in chans]
    ctx = Context(desc)
    alpha = np.linspace(0.0, 1.0, len(chans))
    p, x = _events(ctx, n, 7)
    want = _one_by_one(torch, ctx, range(len(chans)), p, x, alpha)
    for _ in range(2):
        assert torch.equal(ctx.multichannel_density(0, p, x, alpha), want)
    ctx.close()


def _two_processes():
    a, b = W.c2_pp4j(), W.c2_pp4j()
    a["channels"] = a["channels"][:5]
    return {"processes": [a, b]}


def test_captured_density_beside_eager_calls(torch):
    """A captured density of the five-channel process keeps its scratch through
    eager densities of the eight-channel one and of fewer events: every replay
    has the eager call's bits and memory allocated in between is untouched."""
    from paper_2602_06895_amd import Context

    ctx = Context(_two_processes())
    n = 20_003
    al5, al8 = np.full(5, 0.2), np.full(8, 0.125)
    sets = [_events(ctx, n, s) for s in (1, 2, 3)]
    p, x = (t.clone() for t in sets[0])
    eager = [ctx.multichannel_density(0, a, b, al5) for a, b in sets]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = ctx.multichannel_density(0, p, x, al5)
    q, z = _events(ctx, n, 9, chan=5)
    for i in (1, 2, 0, 1):
        want8 = ctx.multichannel_density(1, q, z, al8)
        ctx.multichannel_density(1, q[:, :, :1000].contiguous(), z[:, :1000].contiguous(), al8)
        held = [torch.full((1 << 20,), 3.0, dtype=torch.float64, device="cuda") for _ in range(40)]
        p.copy_(sets[i][0])
        x.copy_(sets[i][1])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager[i])
        assert all(bool((h == 3.0).all()) for h in held)
        assert torch.equal(ctx.multichannel_density(1, q, z, al8), want8)
    del graph
    ctx.close()


def test_density_without_room_for_a_run(torch):
    """With too little memory for eight channels' scratch the density takes one
    at a time, with the same bits, and stays so without allocating again."""
    from paper_2602_06895_amd import Context

    n = 2_700_000  # 238 MB a channel, 1.9 GB for eight
    alpha = np.full(8, 0.125)
    ctx = Context(W.c2_pp4j())
    p, x = _events(ctx, n, 7)
    want = ctx.multichannel_density(0, p, x, alpha)
    ctx.close()
    ctx = Context(W.c2_pp4j())
    ctx.multichannel_density(0, p[:, :, :1000].contiguous(), x[:, :1000].contiguous(), alpha)
    got = torch.empty_like(want)
    torch.cuda.empty_cache()
    hog = []
    try:
        while torch.cuda.mem_get_info()[0] > 1_500_000_000:
            hog.append(torch.empty(512 << 20, dtype=torch.uint8, device="cuda"))
        if torch.cuda.mem_get_info()[0] < 600_000_000:
            pytest.skip("no room for one channel either")

        def call():
            a = np.ascontiguousarray(alpha)
            return ctx.L.msx_multichannel_density(ctx.h, 0, n, p.data_ptr(), x.data_ptr(), a.ctypes.data, got.data_ptr(),
                                                  ctx._stream())

        assert call() == 0, ctx.L.msx_last_error(ctx.h)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    finally:
        hog.clear()
        torch.cuda.empty_cache()
    got.zero_()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    assert call() == 0
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    assert torch.equal(got, want)
    ctx.close()
