"""Captured calls against the CPU oracle: graphs captured on one stream replayed
on two at the same time, beside eager calls on the stream they were captured
on, and after larger calls there have outgrown its workspace."""
import numpy as np
import pytest

import oracle
import paper_1705_08213_amd as ccc
import synth
from gpu_util import assert_ccc_identical, assert_tables_equal, dev, host, say

pytestmark = pytest.mark.gpu


def _outputs(n_v):
    import torch
    P = ccc.n_pairs(n_v)
    return (torch.empty((P, 4), dtype=torch.int32, device="cuda"),
            torch.empty((P, 4), dtype=torch.float64, device="cuda"),
            torch.empty((n_v, 4), dtype=torch.int32, device="cuda"))


def _check(v, n_f, out):
    ot, oc = oracle.two_way(v, n_f)
    assert_tables_equal(host(out[0]), ot)
    assert_ccc_identical(host(out[1]), oc)


def _capture(stream, buf, n_f, out):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        ccc.ccc_2way(buf, n_f, tables=out[0], ccc=out[1], counts=out[2])
    return g


# (n_v, n_f, missing): split fields, whole 32 x 32 tiles, staged tiles
CASES = [(180, 9000, 0.02), (700, 1500, 0.0), (3600, 1100, 0.01)]


def test_graphs_of_one_stream_replayed_together():
    import torch
    cap, side = torch.cuda.Stream(), [torch.cuda.Stream() for _ in CASES]
    vs = [synth.beta_hw(n_v, n_f, seed=6000 + n_v, missing=m) for n_v, n_f, m in CASES]
    bufs = [dev(v) for v in vs]
    outs = [_outputs(n_v) for n_v, _, _ in CASES]
    eager_v = synth.beta_hw(500, 4000, seed=6010, missing=0.03)
    eager = dev(eager_v)
    torch.cuda.synchronize()
    graphs = []
    for (n_v, n_f, _), buf, out in zip(CASES, bufs, outs):
        say("2way capture", n_v, n_f)
        graphs.append(_capture(cap, buf, n_f, out))
    torch.cuda.synchronize()
    for rep in range(4):
        say("replays together", rep)
        for out in outs:
            out[0].zero_()
            out[1].zero_()
        torch.cuda.synchronize()
        for _ in range(3):
            for g, s in zip(graphs, side):
                with torch.cuda.stream(s):
                    g.replay()
            with torch.cuda.stream(cap):
                eager_out = ccc.ccc_2way(eager, 4000)
        torch.cuda.synchronize()
        for v, (_, n_f, _), out in zip(vs, CASES, outs):
            _check(v, n_f, out)
        _check(eager_v, 4000, eager_out)


def test_replays_after_the_stream_outgrew_its_workspace():
    """The larger calls run on the stream that was captured, before each replay,
    on inputs that change between the replays."""
    import torch
    n_v, n_f = 180, 1500
    cap = torch.cuda.Stream()
    inputs = [synth.beta_hw(n_v, n_f, seed=6100 + k, missing=m)
              for k, m in enumerate((0.0, 0.02, 0.0, 0.01))]
    sizes = [(900, 9000), (1500, 9000), (2500, 9000), (3500, 9000)]
    bigs = [dev(synth.beta_hw(a, f, seed=6110 + a, missing=0.01)) for a, f in sizes]
    buf = dev(inputs[0]).clone()
    out = _outputs(n_v)
    torch.cuda.synchronize()
    say("2way capture")
    g = _capture(cap, buf, n_f, out)
    for k, v in enumerate(inputs):
        say("2way replay", k)
        torch.cuda.synchronize()
        with torch.cuda.stream(cap):
            buf.copy_(torch.from_numpy(np.ascontiguousarray(v)))
            ccc.ccc_2way(bigs[k], sizes[k][1])
            out[0].zero_()
            g.replay()
        torch.cuda.synchronize()
        _check(v, n_f, out)


def test_growth_within_one_capture():
    """Two calls of one capture, the second larger: the first one's nodes keep
    their buffer."""
    import torch
    cap = torch.cuda.Stream()
    cases = [(200, 1337, 0.01), (1200, 3000, 0.0)]
    vs = [synth.beta_hw(n_v, n_f, seed=6200 + n_v, missing=m) for n_v, n_f, m in cases]
    bufs = [dev(v) for v in vs]
    outs = [_outputs(n_v) for n_v, _, _ in cases]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=cap):
        for buf, (n_v, n_f, _), out in zip(bufs, cases, outs):
            say("2way capture", n_v, n_f)
            ccc.ccc_2way(buf, n_f, tables=out[0], ccc=out[1], counts=out[2])
    for rep in range(3):
        say("2way replay", rep)
        for out in outs:
            out[0].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ccc.ccc_2way(bufs[1], cases[1][1])
        for v, (_, n_f, _), out in zip(vs, cases, outs):
            _check(v, n_f, out)


def test_destroyed_graphs_give_their_workspaces_back():
    """Forty captures in turn, each destroyed after a replay: the memory that
    the library holds for them does not add up."""
    import torch
    n_v, n_f = 2000, 40000  # 20 MB of operands
    v = synth.beta_hw(n_v, n_f, seed=6300, missing=0.01)
    buf, out = dev(v), _outputs(n_v)
    cap = torch.cuda.Stream()
    ccc.release_workspace()
    ccc.ccc_2way(buf, n_f)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for k in range(40):
        if k % 10 == 0:
            say("2way capture and destroy", k)
        g = _capture(cap, buf, n_f, out)
        g.replay()
        torch.cuda.synchronize()
        del g
        ccc.ccc_2way(buf, n_f)
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] < 15 * 22 * 2**20
    out[0].zero_()
    g = _capture(cap, buf, n_f, out)
    g.replay()
    torch.cuda.synchronize()
    _check(v, n_f, out)
