"""Predictions of one surrogate that overlap: calls on streams that are not
ordered after each other, and calls recorded in a graph whose replays run
beside them.  Each gives the bits of the same call alone: no call sees the
members' outputs of another.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [([5, 64, 64, 1], 5), ([5, 250, 1], 3), ([5, 128, 128, 1], 8), ([5, 256, 256, 256, 1], 5)]


@pytest.fixture(params=SHAPES, ids=str)
def surrogate(gpu, request):
    sde, ctx, dev = gpu
    widths, members = request.param
    s = sde.sde_surrogate_create(ctx, widths, members, 3)
    yield sde, s, dev
    torch.cuda.synchronize()
    sde.sde_surrogate_destroy(s)


def _query(n, seed, dev):
    return torch.from_numpy(np.random.default_rng(seed).uniform(1.0, 5.0, (n, 5)).astype(np.float32)).to(dev)


def _outputs(n, dev):
    return torch.full((2, n), 7.5, device=dev)


@pytest.mark.parametrize("n", [1, 300, 5000])
def test_two_streams(surrogate, n):
    sde, s, dev = surrogate
    X = [_query(n, seed, dev) for seed in range(2)]
    ref = [_outputs(n, dev) for _ in X]
    for x, r in zip(X, ref):
        sde.sde_surrogate_predict(s, x, r[0], r[1])
        torch.cuda.synchronize()
    assert n == 1 or not torch.equal(ref[0], ref[1])
    streams = [torch.cuda.Stream(dev) for _ in X]
    out = [[_outputs(n, dev) for _ in range(20)] for _ in X]
    torch.cuda.synchronize()
    for i in range(20):
        for k, st in enumerate(streams):
            sde.sde_surrogate_predict(s, X[k], out[k][i][0], out[k][i][1], stream=st)
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(o, ref[k]) for o in out[k])


def test_replays_beside_calls(surrogate):
    sde, s, dev = surrogate
    n = 300
    X = [_query(n, seed, dev) for seed in range(2)]
    ref = [_outputs(n, dev) for _ in X]
    for x, r in zip(X, ref):
        sde.sde_surrogate_predict(s, x, r[0], r[1])
    torch.cuda.synchronize()
    out, other = _outputs(n, dev), torch.cuda.Stream(dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sde.sde_surrogate_predict(s, X[0], out[0], out[1])
    for _ in range(4):
        out.fill_(7.5)
        beside = [_outputs(n, dev) for _ in range(3)]
        torch.cuda.synchronize()
        graph.replay()
        for b in beside:
            sde.sde_surrogate_predict(s, X[1], b[0], b[1], stream=other)
        torch.cuda.synchronize()
        assert torch.equal(out, ref[0])
        assert all(torch.equal(b, ref[1]) for b in beside)


def test_null_stream_and_another(surrogate):
    """The null stream orders its own calls without an event: each way from it
    to another stream and back, several calls at a time."""
    sde, s, dev = surrogate
    n = 300
    X = [_query(n, seed, dev) for seed in range(2)]
    ref = [_outputs(n, dev) for _ in X]
    for x, r in zip(X, ref):
        sde.sde_surrogate_predict(s, x, r[0], r[1])
        torch.cuda.synchronize()
    other = torch.cuda.Stream(dev)
    turns = [0, 0, 1, 0, 1, 1, 0, 0, 0, 1, 0, 1] * 3
    out = [_outputs(n, dev) for _ in turns]
    torch.cuda.synchronize()
    for k, o in zip(turns, out):
        sde.sde_surrogate_predict(s, X[k], o[0], o[1], stream=other if k else torch.cuda.default_stream(dev))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref[k]) for k, o in zip(turns, out))
