"""Single calls share the context's pinned staging block: results stay right
across growing and shrinking calls, beside a prepared handle and gcds on the
same context, and after a call that fails."""
import ctypes as C

import numpy as np
import pytest

import paper_1103_4697_amd as snc
import synth
from oracle import resultant as R

pytestmark = pytest.mark.gpu


def test_interleaved_calls_on_one_context():
    ctx = snc.Context(0)
    rng = np.random.default_rng(77)
    pairs = [(synth.dense_bivariate(rng, a, bits=b), synth.dense_bivariate(rng, c, bits=b))
             for a, c, b in [(3, 2, 8), (9, 8, 40), (2, 2, 60), (7, 7, 16)]]
    want = [R.resultant_y(f, g) for f, g in pairs]
    handle = snc.ResultantBatch(pairs, ctx)
    handle.run()
    for _ in range(2):
        for i, (f, g) in enumerate(pairs):
            assert snc.resultant_y(f, g, ctx) == want[i]
            h = [3, -1, 2 + i]
            assert snc.gcd_z(synth.univariate_product(h, [1, 5, 7]), synth.univariate_product(h, [2, -9]), ctx) == h
        assert snc.resultant_y_batch(pairs[::-1], ctx) == want[::-1]
        handle.run()
        assert handle.results() == want
    # an undersized output is refused before any work, and the next call is unaffected
    keep = []
    f, g = pairs[1]
    bf, bg = snc._as_bipoly(f, keep), snc._as_bipoly(g, keep)
    u, _buf = snc._out_upoly(1, 1, keep)
    ws = ctx.workspace(snc.resultant_plan(f, g).workspace_bytes)
    st = snc.lib().snc_resultant_y(ctx.h, C.byref(bf), C.byref(bg), C.c_void_p(ws.data_ptr()), C.c_size_t(ws.numel()),
                                   ctx.stream_handle(), C.byref(u))
    assert st == snc.SNC_ERANGE
    assert snc.resultant_y(*pairs[3], ctx) == want[3]
