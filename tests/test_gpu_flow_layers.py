"""The fused coupling layers (BF16, hidden width 128, up to 16 bins) over the
shapes where their split of the work changes: event counts around a tile of 16
and of 64 events and around one tile per compute unit, one to 32 transformed
coordinates (fewer than, as many as, and more than a workgroup's waves), bin
counts with and without padding."""
import numpy as np
import pytest

import workloads as W
from oracle import flow as F

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t

    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


def _pair(d, layers, bins, seed, scale=0.05):
    import torch as t

    from paper_2602_06895_amd import FLOW_BF16, Flow

    params = W.flow_params(seed, d, layers, bins, 128, last_scale=scale)
    f = Flow(d, layers, bins, 128, mlp=FLOW_BF16)
    f.set_params(params)
    return f, F.Flow(d, layers, bins, 128, params=t.as_tensor(params.astype(np.float64)), bf16_mlp=True)


SHAPES = [(16, 5, 16, 1), (16, 4, 16, 15), (16, 4, 16, 16), (16, 4, 16, 17), (10, 4, 16, 1000), (16, 2, 16, 4096),
          (16, 2, 16, 4097), (14, 2, 16, 16385), (2, 3, 16, 100), (18, 2, 16, 4200), (64, 2, 16, 300),
          (64, 2, 12, 4160), (16, 4, 1, 70), (16, 2, 2, 5000), (10, 2, 15, 70), (18, 2, 5, 90),
          (10, 4, 8, 1000), (16, 2, 8, 4097), (64, 2, 8, 300)]


@pytest.mark.parametrize("d,layers,bins,n", SHAPES)
def test_passes_match_oracle(torch, d, layers, bins, n):
    """Forward and inverse against the oracle with BF16 conditioner roundings;
    bounds: one BF16 rounding decision taken the other way on an FP32
    accumulator, as for the full-size flows."""
    f, orc = _pair(d, layers, bins, 10 * d + bins)
    u = W.philox_uniforms_f32(3, d, 0, n, d)
    t = torch.from_numpy(u).cuda()
    y, ld = f.forward(t)
    x, lq = f.inverse(t)
    torch.cuda.synchronize()
    ref = torch.from_numpy(u.T.astype(np.float64))
    for got, gl, (want, wl) in ((y, ld, orc.forward(ref)), (x, lq, orc.inverse(ref))):
        assert np.abs(got.cpu().numpy().T - want.numpy()).max() < 2e-3
        assert np.abs(gl.cpu().numpy() - wl.numpy()).max() < 2e-2
    f.close()


@pytest.mark.parametrize("d,n", [(16, 100), (16, 9001), (24, 5000)])
def test_passes_in_place_and_split(torch, d, n):
    """A pass over its own buffer, and over the two halves of a batch: the same
    bits (no event meets another)."""
    f, _ = _pair(d, 5, 16, 77)
    u = torch.from_numpy(W.philox_uniforms_f32(4, 1, 0, n, d)).cuda()
    for name in ("forward", "inverse"):
        v, ld = getattr(f, name)(u)
        w, lw = u.clone(), torch.empty(n, dtype=torch.float32, device="cuda")
        f._check(getattr(f.L, "msx_flow_" + name)(f.h, n, w.data_ptr(), w.data_ptr(), lw.data_ptr(), f._stream()))
        assert torch.equal(w, v) and torch.equal(lw, ld)
        k = n // 2 + 3
        parts = [getattr(f, name)(p.contiguous()) for p in (u[:, :k], u[:, k:])]
        assert torch.equal(torch.cat([p[0] for p in parts], 1), v)
        assert torch.equal(torch.cat([p[1] for p in parts]), ld)
    f.close()


def _batch(torch, d, n, seed):
    rng = np.random.default_rng(seed)
    y = rng.uniform(0.02, 0.98, (d, n)).astype(np.float32)
    wfj = rng.uniform(0.5, 2.0, n)
    lqo = rng.uniform(-0.5, 0.5, n).astype(np.float32)
    return y, wfj, lqo, [torch.from_numpy(a).cuda() for a in (y, wfj, lqo)]


# one event, around a tile, an odd number of 32-event blocks per run of the
# weight gradients, up to and beyond one tile of 32 per compute unit and the
# largest number of runs
GRAD_SHAPES = [(16, 4, 16, 1), (16, 4, 16, 63), (16, 3, 16, 65), (10, 4, 16, 513), (2, 3, 16, 200), (16, 2, 16, 2100),
               (18, 2, 16, 130), (64, 2, 16, 70), (64, 2, 12, 300), (16, 4, 1, 90), (14, 2, 7, 33000), (24, 2, 5, 700)]


@pytest.mark.parametrize("d,layers,bins,n", GRAD_SHAPES)
def test_gradient_matches_oracle(torch, d, layers, bins, n):
    """The gradient against the oracle with BF16 conditioner roundings.  That
    oracle differs from the FP64 one by d_bf16; the kernels round the same
    quantities, but from FP32 sums, and the back-propagated ones too, each worth
    at most one more such rounding: 2 d_bf16 + 1e-3, as for the full-size flow."""
    import torch as t

    f, orc = _pair(d, layers, bins, 7 * d + bins)
    y, wfj, lqo, dev = _batch(torch, d, n, d + n)
    g, loss = f.gradient(*dev)
    torch.cuda.synchronize()
    args = [t.from_numpy(y.T.astype(np.float64)), t.from_numpy(wfj) ** 2, t.from_numpy(lqo.astype(np.float64))]
    l_bf, g_bf = orc.loss_and_grad(*args)
    _, g_64 = F.Flow(d, layers, bins, 128, params=orc.params, bf16_mlp=False).loss_and_grad(*args)
    got, ref, ref64 = g.cpu().numpy().astype(np.float64), g_bf.numpy(), g_64.numpy()
    bound = 2 * np.linalg.norm(ref - ref64) + 1e-3 * np.linalg.norm(ref)
    assert np.linalg.norm(got - ref) <= bound
    assert abs(float(loss.cpu()[0]) - float(l_bf)) <= 1e-3 * abs(float(l_bf))
    f.close()


@pytest.mark.parametrize("d,bins", [(16, 16), (24, 9)])
def test_gradient_after_a_larger_batch(torch, d, bins):
    """A batch that is no whole tile, in the buffers of a larger one: the bits of
    a flow that has seen nothing else."""
    f, _ = _pair(d, 3, bins, 5)
    *_, big = _batch(torch, d, 3000, 1)
    *_, small = _batch(torch, d, 77, 2)
    want, _ = f.gradient(*small)
    f.gradient(*big)
    got, _ = f.gradient(*small)
    assert torch.equal(got, want)
    f.close()


def _pair_f32(d, layers, bins, seed):
    import torch as t

    from paper_2602_06895_amd import FLOW_FP32, Flow

    params = W.flow_params(seed, d, layers, bins, 128, last_scale=0.05)
    f = Flow(d, layers, bins, 128, mlp=FLOW_FP32)
    f.set_params(params)
    return f, F.Flow(d, layers, bins, 128, params=t.as_tensor(params.astype(np.float64)), bf16_mlp=False)


# tiles of 16, 32 and 64 events, up to and beyond one per compute unit
@pytest.mark.parametrize("d,layers,bins,n", [(16, 3, 16, 1), (16, 4, 16, 33), (2, 3, 16, 100), (10, 4, 16, 4096),
                                             (16, 2, 16, 4097), (16, 2, 16, 8200), (18, 2, 5, 90), (64, 2, 12, 300),
                                             (16, 4, 1, 70), (14, 2, 16, 16500)])
def test_fp32_passes_match_oracle(torch, d, layers, bins, n):
    """FP32 conditioners against the FP64 oracle, with the bounds of the full-size
    flows (a few hundred roundings of 6e-8 through up to as many layers)."""
    f, orc = _pair_f32(d, layers, bins, 10 * d + bins)
    u = W.philox_uniforms_f32(3, d, 0, n, d)
    t = torch.from_numpy(u).cuda()
    y, ld = f.forward(t)
    x, lq = f.inverse(t)
    torch.cuda.synchronize()
    ref = torch.from_numpy(u.T.astype(np.float64))
    for got, gl, (want, wl) in ((y, ld, orc.forward(ref)), (x, lq, orc.inverse(ref))):
        assert np.abs(got.cpu().numpy().T - want.numpy()).max() < 2e-5
        assert np.abs(gl.cpu().numpy() - wl.numpy()).max() < 2e-4
    f.close()


@pytest.mark.parametrize("d,layers,bins,n", [(16, 4, 16, 1), (16, 4, 16, 31), (16, 3, 16, 65), (10, 4, 16, 513),
                                             (2, 3, 16, 200), (16, 2, 16, 2100), (18, 2, 16, 130), (64, 2, 12, 300),
                                             (16, 4, 1, 90), (24, 2, 5, 700)])
def test_fp32_gradient_matches_oracle(torch, d, layers, bins, n):
    """The FP32 gradient against the FP64 oracle, with the bound of the full-size
    flow; a step afterwards leaves operands that give the same density as the
    parameters read back into a new flow."""
    import torch as t

    from paper_2602_06895_amd import FLOW_FP32, Flow

    f, orc = _pair_f32(d, layers, bins, 7 * d + bins)
    y, wfj, lqo, dev = _batch(torch, d, n, d + n)
    g, loss = f.gradient(*dev)
    torch.cuda.synchronize()
    l_ref, ref = orc.loss_and_grad(t.from_numpy(y.T.astype(np.float64)), t.from_numpy(wfj) ** 2,
                                   t.from_numpy(lqo.astype(np.float64)))
    got, ref = g.cpu().numpy().astype(np.float64), ref.numpy()
    assert np.linalg.norm(got - ref) <= 1e-3 * np.linalg.norm(ref)
    assert abs(float(loss.cpu()[0]) - float(l_ref)) <= 1e-4 * abs(float(l_ref))
    f.train_step(*dev, lr=1e-3)
    h = Flow(d, layers, bins, 128, mlp=FLOW_FP32)
    h.set_params(f.get_params())
    for a, b in zip(f.inverse(dev[0]), h.inverse(dev[0])):
        assert torch.equal(a, b)
    f.close()
    h.close()


@pytest.mark.parametrize("d,bins,n", [(16, 16, 1 << 18), (10, 8, 1 << 16), (18, 5, 1 << 15)])
def test_fp32_gradient_sums_stay_short(torch, d, bins, n):
    """n equal events, n a power of two: every event adds the same term, the
    one-event gradient divided by n exactly, so the sum should be that gradient.
    An accumulator takes one run of at most max(256, n / 512) events, a rounding
    each, and the partial sums of up to 512 runs are added in 16 chains: (run +
    40) u relative, whatever n is."""
    f, _ = _pair_f32(d, 2, bins, 3)
    *_, one = _batch(torch, d, 1, 4)
    want, _ = f.gradient(*one)
    got, _ = f.gradient(one[0].expand(d, n).contiguous(), one[1].expand(n).contiguous(), one[2].expand(n).contiguous())
    err = (got.double() - want.double()).abs()
    assert bool((err <= (max(256, n // 512) + 40) * 2.0 ** -24 * want.double().abs() + 1e-30).all())
    f.close()


def test_fp32_gradient_blocks_of_a_large_batch(torch):
    """Every weight and bias gradient of its own against the FP64 oracle, at more
    events than the number of runs is limited by; the bound of the whole
    gradient."""
    import torch as t

    d, layers, bins, n = 16, 2, 16, 40_001
    f, orc = _pair_f32(d, layers, bins, 11)
    y, wfj, lqo, dev = _batch(torch, d, n, 12)
    g, _ = f.gradient(*dev)
    _, ref = orc.loss_and_grad(t.from_numpy(y.T.astype(np.float64)), t.from_numpy(wfj) ** 2,
                               t.from_numpy(lqo.astype(np.float64)))
    got, ref = g.cpu().numpy().astype(np.float64), ref.numpy()
    at = 0
    for _ in range(layers):
        for shape in orc.shapes:
            k = int(np.prod(shape))
            assert np.linalg.norm(got[at:at + k] - ref[at:at + k]) <= 1e-3 * np.linalg.norm(ref[at:at + k])
            at += k
    f.close()


@pytest.mark.parametrize("d", [10, 16])
@pytest.mark.parametrize("bins", range(1, 17))
def test_small_and_large_passes_agree(torch, d, bins):
    """A pass in tiles of 16 events and one in tiles of 64: the same bits for every
    number of bins."""
    f, _ = _pair(d, 4, bins, 3)
    u = torch.from_numpy(W.philox_uniforms_f32(3, 1, 0, 5000, d)).cuda()
    for name in ("inverse", "forward"):
        large, small = getattr(f, name)(u), getattr(f, name)(u[:, :1000].contiguous())
        assert torch.equal(small[0], large[0][:, :1000]) and torch.equal(small[1], large[1][:1000])
    f.close()


def _reverse_edge(torch):
    """The largest batch whose reverse kernels take tiles of 32 events: one for
    every compute unit."""
    return 32 * torch.cuda.get_device_properties(0).multi_processor_count


# up to the edge tiles of 32 events, beyond it of 64: 16 and fewer bins, one and
# more chunks of eight coordinates, a partial last tile
@pytest.mark.parametrize("d,layers,bins,beyond", [(16, 2, 16, 0), (16, 2, 16, 1), (16, 2, 16, 107), (18, 2, 16, 75),
                                                  (24, 2, 5, 97), (64, 2, 12, 33), (64, 1, 16, 65), (10, 2, 8, 64),
                                                  (2, 2, 16, 31)])
def test_gradient_around_the_tile_edge(torch, d, layers, bins, beyond):
    """The gradient of batches at and beyond the edge against the oracle, with the
    bound of the other shapes."""
    test_gradient_matches_oracle(torch, d, layers, bins, _reverse_edge(torch) + beyond)


@pytest.mark.parametrize("d,bins", [(16, 16), (24, 9)])
def test_gradient_across_the_tile_edge(torch, d, bins):
    """Batches of both tile sizes in turn in the same buffers: the bits of a flow
    that has seen nothing else."""
    sizes = [_reverse_edge(torch) + 523, 77, _reverse_edge(torch) + 40, _reverse_edge(torch) - 1]
    f, _ = _pair(d, 3, bins, 5)
    for n in sizes:
        *_, dev = _batch(torch, d, n, n)
        got, _ = f.gradient(*dev)
        h, _ = _pair(d, 3, bins, 5)
        want, _ = h.gradient(*dev)
        assert torch.equal(got, want)
        h.close()
    f.close()
