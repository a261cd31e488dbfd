"""Multi-allelic outputs of every number of states around the 16-row blocks and
the tiles, with tables alone, CCC alone and both, against the CPU oracle:
entries that are not the call's keep what they held."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_1705_08213_amd as ccc
import synth
from gpu_util import assert_ccc_identical, assert_tables_equal, dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [2, 3, 4])
@pytest.mark.parametrize("n_v,n_f", [(2, 130), (15, 1), (17, 127), (33, 129), (64, 300), (97, 128)])
def test_multi_outputs_around_the_tiles(s, n_v, n_f):
    import torch
    v = synth.multi_hw(n_v, n_f, s, seed=6400 + n_v, missing=0.05)
    ot, oc = oracle.multi_two_way(v, n_f, s)
    dv, P, ss = dev(v), ccc.n_pairs(n_v), s * s
    for tables, values in ((True, True), (True, False), (False, True)):
        say("multi outputs", s, n_v, n_f, tables, values)
        # one entry more at the end, which no call may touch
        t = torch.full((P + 1, ss), -7, dtype=torch.int32, device="cuda")
        c = torch.full((P + 1, ss), -7.0, dtype=torch.float64, device="cuda")
        o = ccc.make_opts("mfma", operands="fp4")
        st = ccc.lib().ccc_2way_multi(dv.data_ptr(), n_v, n_f, v.shape[1], s,
                                      t.data_ptr() if tables else None,
                                      c.data_ptr() if values else None, None, ctypes.byref(o),
                                      torch.cuda.current_stream().cuda_stream)
        assert st == ccc.CCC_OK
        torch.cuda.synchronize()
        t, c = host(t), host(c)
        assert (t[P] == -7).all() and (c[P] == -7.0).all()
        if tables:
            assert_tables_equal(t[:P], ot)
        else:
            assert (t == -7).all()
        if values:
            assert_ccc_identical(c[:P], oc)
        else:
            assert (c == -7.0).all()
