"""Every form of a 2-way call on every tile shape, on operands and on packed
rows, against the CPU oracle: row ranges that begin and end inside tiles,
selections, accumulating blocks, streamed tables at ragged sizes, batches, and
the largest sums that the shapes hold exactly."""
import numpy as np
import pytest

import oracle
import paper_1705_08213_amd as ccc
import synth
from gpu_util import assert_ccc_identical, assert_tables_equal, dev, host, say

pytestmark = pytest.mark.gpu

# (shape, splits, operand limit): 64 x 128 staged, 64 x 64 staged, 32 x 32
# field-split by one and three workgroups; on packed rows 128 x 64 (with its
# cooperative complete form), 64 x 32, 64 x 64
ROUTES = [("0", "", ""), ("2", "", ""), ("1", "1", ""), ("1", "3", ""),
          ("0", "", "0"), ("1", "", "0"), ("2", "", "0")]


@pytest.fixture(params=ROUTES, ids=["-".join(r) for r in ROUTES])
def route(request, monkeypatch):
    shape, split, limit = request.param
    monkeypatch.setenv("CCC_ONESHOT_VARIANT", shape)
    if split:
        monkeypatch.setenv("CCC_SPLIT", split)
    if limit:
        monkeypatch.setenv("CCC_OPERAND_LIMIT", limit)
    return request.param


_wanted = {}


def _triangle(n_v, n_f, missing):
    key = (n_v, n_f, missing)
    if key not in _wanted:
        v = synth.beta_hw(n_v, n_f, seed=7000 + n_v, missing=missing)
        _wanted[key] = (v, *oracle.two_way(v, n_f))
    return _wanted[key]


def _pair0(n, i):
    """Index of the first pair of row i."""
    return i * n - i * (i + 1) // 2


# ranges inside one tile, over the edges of the 32, 64, 128 and 256 row tiles,
# and to the last rows
RANGES = [(0, 1), (100, 130), (130, 390), (255, 257), (256, 600), (511, 700), (640, 699), (698, 700)]


@pytest.mark.parametrize("missing", [0.0, 0.03])
def test_row_ranges(route, missing):
    n_v, n_f = 700, 300
    v, ot, oc = _triangle(n_v, n_f, missing)
    dv = dev(v)
    for lo, hi in RANGES:
        say("2way rows", route, missing, lo, hi)
        t, c, cnt = ccc.ccc_2way_rows(dv, n_f, lo, hi)
        p0, p1 = _pair0(n_v, lo), _pair0(n_v, hi)
        assert_tables_equal(host(t), ot[p0:p1])
        assert_ccc_identical(host(c), oc[p0:p1])
        m = host(cnt)  # of every row, also those before the range
        assert (m[:, 0] + m[:, 1] == 2 * m[:, 2]).all() and (m[:, 2] >= n_f * (0.8 if missing else 1)).all()


@pytest.mark.parametrize("missing", [0.0, 0.03])
def test_selections(route, missing):
    n_v, n_f = 700, 300
    v, ot, oc = _triangle(n_v, n_f, missing)
    threshold = float(np.quantile(oc.max(axis=1), 0.9))
    want = np.flatnonzero((oc >= threshold).any(axis=1))
    say("2way select", route, missing, len(want))
    n, index, c, t = ccc.ccc_2way_select(dev(v), n_f, threshold, len(want) + 10)
    assert n == len(want)
    order = np.argsort(host(index))
    assert np.array_equal(host(index)[order], want)
    assert_ccc_identical(host(c)[order], oc[want])
    assert_tables_equal(host(t)[order], ot[want])


@pytest.mark.parametrize("missing", [0.0, 0.03])
@pytest.mark.parametrize("n_a,n_b", [(333, 290), (129, 257), (31, 1), (1, 300)])
def test_blocks_whole_and_in_chunks(route, missing, n_a, n_b):
    import torch
    n_f, chunk = 900, 512
    va = synth.beta_hw(n_a, n_f, seed=7100 + n_a, missing=missing)
    vb = synth.beta_hw(n_b, n_f, seed=7200 + n_b, missing=missing)
    ot, oc = oracle.block(va, vb, n_f)
    da, db = dev(va), dev(vb)
    for chunks in ([(0, n_f)], [(0, chunk), (chunk, n_f - chunk)]):
        say("2way block", route, missing, n_a, n_b, len(chunks))
        t = torch.full((n_a, n_b, 4), -1, dtype=torch.int32, device="cuda")
        c = torch.full((n_a, n_b, 4), -1.0, dtype=torch.float64, device="cuda")
        ca = torch.full((n_a, 4), -1, dtype=torch.int32, device="cuda")
        cb = torch.full((n_b, 4), -1, dtype=torch.int32, device="cuda")
        for k, (f0, m) in enumerate(chunks):
            last = k == len(chunks) - 1
            ccc.ccc_2way_block(da, db, m, t, ca, cb, c if last else None, accumulate=k > 0,
                               finalize=last, field_offset=f0 // 4)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)


@pytest.mark.parametrize("shape", ["0", "2"])
def test_streamed_tables_at_ragged_sizes(shape, monkeypatch):
    """Complete data on both sides of the lines from which tables are streamed."""
    import torch
    monkeypatch.setenv("CCC_ONESHOT_VARIANT", shape)
    for n_v, n_f in ((257, 12287), (257, 12288), (131, 12545)):
        say("2way complete", shape, n_v, n_f)
        v, ot, oc = _triangle(n_v, n_f, 0.0)
        t, c, _ = ccc.ccc_2way(dev(v), n_f)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)
    for n_a, n_b, n_f in ((130, 260, 2999), (130, 260, 3000), (70, 516, 3073), (130, 261, 3073)):
        say("2way complete block", shape, n_a, n_b, n_f)
        va = synth.beta_hw(n_a, n_f, seed=7300 + n_a, missing=0.0)
        vb = synth.beta_hw(n_b, n_f, seed=7400 + n_b, missing=0.0)
        ot, oc = oracle.block(va, vb, n_f)
        t = torch.empty((n_a, n_b, 4), dtype=torch.int32, device="cuda")
        c = torch.empty((n_a, n_b, 4), dtype=torch.float64, device="cuda")
        ca = torch.empty((n_a, 4), dtype=torch.int32, device="cuda")
        cb = torch.empty((n_b, 4), dtype=torch.int32, device="cuda")
        ccc.ccc_2way_block(dev(va), dev(vb), n_f, t, ca, cb, c)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)


def _extremes(n_f, seed):
    """Rows all missing (the largest sum of the code plane, 9 n_f), all 11, all
    00, and random ones."""
    const = synth.constant([2, 2, 3, 3, 0], n_f, seed=seed)
    return np.ascontiguousarray(np.concatenate([const, synth.beta_hw(3, n_f, seed=seed,
                                                                     missing=0.02)]))


STAGED_MOST = ((1 << 24) - 1) // 9  # 9 n_f < 2^24


@pytest.mark.parametrize("shape", ["0", "1", "2"])
@pytest.mark.parametrize("n_f", [STAGED_MOST, STAGED_MOST + 1])
def test_largest_sums_of_the_staged_tiles(shape, n_f, monkeypatch):
    monkeypatch.setenv("CCC_ONESHOT_VARIANT", shape)
    say("largest sums", shape, n_f)
    v = _extremes(n_f, seed=11)
    t, c, _ = ccc.ccc_2way(dev(v), n_f)
    ot, oc = oracle.two_way(v, n_f)
    assert_tables_equal(host(t), ot)
    assert_ccc_identical(host(c), oc)


@pytest.mark.parametrize("shape", ["0", "1", "2"])
@pytest.mark.parametrize("n_f", [(1 << 22) - 1, 1 << 22])
def test_largest_sums_on_packed_rows(shape, n_f, monkeypatch):
    """The packed form's sums of U = rho(1) + 2 [missing] reach 4 n_f = 2^24."""
    monkeypatch.setenv("CCC_ONESHOT_VARIANT", shape)
    monkeypatch.setenv("CCC_OPERAND_LIMIT", "0")
    say("largest sums on packed rows", shape, n_f)
    for v in (_extremes(n_f, seed=12),
              np.ascontiguousarray(np.concatenate([synth.constant([3, 3, 0, 1], n_f, seed=13),
                                                   synth.beta_hw(2, n_f, seed=14, missing=0.0)]))):
        t, c, _ = ccc.ccc_2way(dev(v), n_f)
        ot, oc = oracle.two_way(v, n_f)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)


@pytest.mark.parametrize("variant", ["", "0", "1", "2", "3"])
def test_batches_on_packed_rows(variant, monkeypatch):
    monkeypatch.setenv("CCC_OPERAND_LIMIT", "0")
    if variant:
        monkeypatch.setenv("CCC_MANY_VARIANT", variant)
    sizes = [(1, 100, 0.0), (33, 257, 0.03), (300, 1000, 0.0), (129, 513, 0.02), (64, 2049, 1.0)]
    vs = [synth.beta_hw(n_v, n_f, seed=7500 + n_v, missing=m) for n_v, n_f, m in sizes]
    say("2way many packed", variant)
    outs = ccc.ccc_2way_many([dict(v=dev(v), n_f=n_f) for v, (_, n_f, _) in zip(vs, sizes)])
    for v, (n_v, n_f, _), (t, c, _) in zip(vs, sizes, outs):
        if n_v < 2:
            continue
        ot, oc = oracle.two_way(v, n_f)
        assert_tables_equal(host(t), ot)
        assert_ccc_identical(host(c), oc)


def test_batch_with_a_large_problem_on_long_fields():
    """A problem of 3000 tiles and more past the staged tiles' fields takes the
    whole batch to the packed rows; beside it a small one."""
    n_f = STAGED_MOST + 1
    small = synth.beta_hw(200, 700, seed=7600, missing=0.02)
    base = _extremes(n_f, seed=15)
    rows = np.arange(2480) % base.shape[0]
    say("2way many long fields")
    big = dev(base)[dev(rows.astype(np.int64))].contiguous()
    (t, _, _), (ts, cs, _) = ccc.ccc_2way_many([dict(v=big, n_f=n_f, want_ccc=False),
                                                dict(v=dev(small), n_f=700)])
    ot, oc = oracle.two_way(small, 700)
    assert_tables_equal(host(ts), ot)
    assert_ccc_identical(host(cs), oc)
    # every pair of the large one is a pair of base rows
    n, k = 2480, base.shape[0]
    pt = np.zeros((k, k, 4), dtype=np.int64)
    bt, _ = oracle.block(base, base, n_f)
    pt[:] = bt.reshape(k, k, 4)
    got = host(t)
    for i in list(range(0, n - 1, 97)) + [31, 32, 63, 64, 127, 128, 2477, 2478]:
        p = _pair0(n, i)
        assert_tables_equal(got[p:p + n - 1 - i], pt[i % k][np.arange(i + 1, n) % k])


@pytest.mark.parametrize("limit", ["", "0"])
@pytest.mark.parametrize("shift", [0, 100])
def test_blocks_whose_sides_share_counts(shift, limit, monkeypatch):
    """Both sides are rows of one set and point into one array of counts; an
    accumulating call adds both sides' counts to the shared entries."""
    import torch
    if limit:
        monkeypatch.setenv("CCC_OPERAND_LIMIT", limit)
    n, n_f, chunk = 300, 900, 512
    m = n - shift
    v = synth.beta_hw(n, n_f, seed=7700, missing=0.02)
    dv = dev(v)
    va, vb = dv[:m].contiguous(), dv[shift:].contiguous()
    counts = torch.zeros((n, 4), dtype=torch.int32, device="cuda")
    t = torch.zeros((m, m, 4), dtype=torch.int32, device="cuda")
    say("2way block shared counts", shift, limit)
    for f0, k in ((0, chunk), (chunk, n_f - chunk)):
        ccc.ccc_2way_block(va, vb, k, t, counts[:m], counts[shift:], accumulate=True,
                           finalize=False, field_offset=f0 // 4)
    ot, _ = oracle.block(v[:m], v[shift:], n_f)
    assert_tables_equal(host(t), ot)
    _, _, one = ccc.ccc_2way(dv, n_f)
    want = host(one)
    times = np.zeros(n, dtype=np.int64)
    times[:m] += 1
    times[shift:] += 1
    assert np.array_equal(host(counts), want * times[:, None])


@pytest.mark.parametrize("complete", [False, True])
def test_large_call_on_long_fields(complete):
    """3000 tiles past the staged tiles' fields: the packed rows' kernel, or the
    one-plane tiles of complete data with the largest sums (rows all 11)."""
    n_f, n = STAGED_MOST + 1, 2480
    base = _extremes(n_f, seed=16)
    if complete:
        base = np.ascontiguousarray(np.concatenate([
            synth.constant([3, 3, 0, 1], n_f, seed=17),
            synth.beta_hw(3, n_f, seed=18, missing=0.0)]))
    k = base.shape[0]
    say("2way long fields", complete)
    big = dev(base)[dev((np.arange(n) % k).astype(np.int64))].contiguous()
    t, c, _ = ccc.ccc_2way(big, n_f)
    bt, bc = oracle.block(base, base, n_f)
    bt, bc = bt.reshape(k, k, 4), bc.reshape(k, k, 4)
    t, c = host(t), host(c)
    for i in list(range(0, n - 1, 97)) + [31, 32, 63, 64, 127, 128, 255, 256, 2477, 2478]:
        p, js = _pair0(n, i), np.arange(i + 1, n) % k
        assert_tables_equal(t[p:p + n - 1 - i], bt[i % k][js])
        assert_ccc_identical(c[p:p + n - 1 - i], bc[i % k][js])
