"""The 2-way kernels on pre-laid operands against the CPU oracle at the edges of
their tiles, shares and dispatch: every tile shape, field splits, long rows in
shares, the packed-row route when the operands find no room, and calls on two
streams and under graph capture, whose operands must not be shared."""
import numpy as np
import pytest

import oracle
import paper_1705_08213_amd as ccc
import synth
from gpu_util import assert_ccc_identical, assert_tables_equal, dev, host, say

pytestmark = pytest.mark.gpu


def _check(v, n_f, out):
    t, c, n = out
    ot, oc = oracle.two_way(v, n_f)
    assert_tables_equal(host(t), ot)
    assert_ccc_identical(host(c), oc)
    m = host(n)
    assert (m[:, 0] + m[:, 1] == 2 * m[:, 2]).all()


# (n_v, n_f): one short of, at and past the 32-, 64- and 128-row tiles, the
# 128-field halves and the 256-field super-steps
SIZES = [(31, 255), (32, 256), (33, 257), (65, 129), (129, 513), (257, 1), (140, 2049)]


@pytest.mark.parametrize("missing", [0.0, 0.03, 1.0])
@pytest.mark.parametrize("variant,split", [("0", ""), ("2", ""), ("1", "1"), ("1", "3"), ("1", "7")])
def test_every_tile_shape(variant, split, missing, monkeypatch):
    monkeypatch.setenv("CCC_ONESHOT_VARIANT", variant)
    if split:
        monkeypatch.setenv("CCC_SPLIT", split)
    for n_v, n_f in SIZES:
        say("2way operands", variant, split, missing, n_v, n_f)
        v = synth.beta_hw(n_v, n_f, seed=5000 + n_v, missing=missing)
        _check(v, n_f, ccc.ccc_2way(dev(v), n_f, path="mfma", operands="fp4"))


@pytest.mark.parametrize("n_v,n_f,missing", [(17, 66000, 0.02), (40, 70001, 0.0), (3, 65536, 0.5)])
def test_long_rows_in_shares(n_v, n_f, missing):
    say("2way shares", n_v, n_f, missing)
    v = synth.beta_hw(n_v, n_f, seed=5100 + n_v, missing=missing)
    _check(v, n_f, ccc.ccc_2way(dev(v), n_f))


@pytest.mark.parametrize("limit", ["0", "100000"])
def test_packed_rows_when_operands_find_no_room(limit, monkeypatch):
    monkeypatch.setenv("CCC_OPERAND_LIMIT", limit)
    for n_v, n_f, missing in ((150, 1100, 0.02), (300, 2050, 0.0)):
        say("2way packed", limit, n_v, n_f)
        v = synth.beta_hw(n_v, n_f, seed=5200 + n_v, missing=missing)
        _check(v, n_f, ccc.ccc_2way(dev(v), n_f))


def test_calls_on_two_streams():
    """Interleaved calls on two streams, nothing ordered between them."""
    import torch
    vs = [synth.beta_hw(400, 3000 + 300 * k, seed=5300 + k, missing=0.01 * k) for k in range(2)]
    ds = [dev(v) for v in vs]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    outs = [[], []]
    for rep in range(6):
        for k in range(2):
            say("2way streams", rep, k)
            with torch.cuda.stream(streams[k]):
                outs[k].append(ccc.ccc_2way(ds[k], 3000 + 300 * k))
    torch.cuda.synchronize()
    for k in range(2):
        for out in outs[k]:
            _check(vs[k], 3000 + 300 * k, out)


def test_capture_keeps_its_workspace():
    """A captured call replays correctly after larger eager calls have grown
    the workspaces, on inputs that change between the replays."""
    import torch
    n_v, n_f = 180, 1500
    inputs = [synth.beta_hw(n_v, n_f, seed=5400 + k, missing=m)
              for k, m in enumerate((0.0, 0.02, 0.0))]
    buf = dev(inputs[0]).clone()
    tables = torch.empty((ccc.n_pairs(n_v), 4), dtype=torch.int32, device="cuda")
    values = torch.empty((ccc.n_pairs(n_v), 4), dtype=torch.float64, device="cuda")
    counts = torch.empty((n_v, 4), dtype=torch.int32, device="cuda")
    big = dev(synth.beta_hw(900, 9000, seed=5410, missing=0.01))
    ccc.ccc_2way(buf, n_f, tables=tables, ccc=values, counts=counts)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    say("2way capture")
    with torch.cuda.graph(g):
        ccc.ccc_2way(buf, n_f, tables=tables, ccc=values, counts=counts)
    for k, v in enumerate(inputs):
        say("2way replay", k)
        buf.copy_(torch.from_numpy(np.ascontiguousarray(v)))
        ccc.ccc_2way(big, 9000)
        tables.zero_()
        g.replay()
        torch.cuda.synchronize()
        _check(v, n_f, (tables, values, counts))


@pytest.mark.parametrize("limit", ["", "0"])
@pytest.mark.parametrize("s", [2, 3, 4])
def test_multi_allelic_on_operands(s, limit, monkeypatch):
    """Both routes of the multi-allelic call around its 128-field steps and
    its tiles."""
    if limit:
        monkeypatch.setenv("CCC_OPERAND_LIMIT", limit)
    for n_v, n_f, missing in ((2, 1, 0.0), (33, 127, 0.02), (65, 128, 0.3), (97, 129, 0.0),
                              (130, 5000, 0.01), (64, 9000, 1.0)):
        say("multi operands", s, limit, n_v, n_f)
        v = synth.multi_hw(n_v, n_f, s, seed=5500 + n_v, missing=missing)
        t, c, _ = ccc.ccc_2way_multi(dev(v), n_f, s)
        ot, oc = oracle.multi_two_way(v, n_f, s)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)


@pytest.mark.parametrize("n_v,n_f", [(225, 40), (257, 300), (289, 90)])
def test_3way_complete_data_around_the_small_call_rule(n_v, n_f):
    """Complete inputs on both sides of the unit count at which the 3-way call
    takes its complete-data form, with and without one missing entry."""
    v = synth.beta_hw(n_v, n_f, seed=5600 + n_v, missing=0.0)
    for k in range(2):
        if k:
            v = v.copy()
            v[n_v // 2, 0] = (v[n_v // 2, 0] & 0xFC) | 2
        say("3way small rule", n_v, n_f, k)
        t, c, _ = ccc.ccc_3way(dev(v), n_f)
        ot, oc = oracle.three_way(v, n_f)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)
