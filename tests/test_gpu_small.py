"""GPU tests of the small-instance kernel (n <= 192, the whole run in one
workgroup's LDS): byte-identical to the CPU oracle at the edges of its rows per
lane, on ties, negative and subnormal values; the caller's matrix is left as it
was, rejected input leaves the records as they were."""
import numpy as np
import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    with hac.Context(0) as c:
        yield c


@pytest.mark.parametrize("n", [2, 3, 4, 17, 63, 64, 65, 127, 128, 129, 144, 145, 191, 192, 193])
def test_small_matches_oracle(ctx, n):
    import torch
    for name, d in (("mixture", synth.mixture_8192(seed=n, n=n)), ("quantized", synth.quantized_matrix(n, n, levels=3)),
                    ("constant", np.full((n, n), 2.5, np.float32)), ("negative", synth.uniform_matrix(n, n, -1.0, 1.0)),
                    ("subnormal", synth.uniform_matrix(n, n) * np.float32(1e-38))):
        t = torch.from_numpy(np.ascontiguousarray(d)).cuda()
        for link in hac.LINKAGES:
            print("small: %s n=%d %s" % (name, n, link), flush=True)
            got = ctx.run(t, link, preserve=True)
            assert got.tobytes() == oracle.run_f32(d, link).tobytes()
        assert torch.equal(t.cpu(), torch.from_numpy(np.ascontiguousarray(d)))


def test_small_input_conventions(ctx):
    import ctypes
    import torch
    d = synth.quantized_matrix(150, 4)
    d[3, 10] = -0.0
    junk = d.copy()
    junk[np.tril_indices(150, 0)] = np.nan
    exp = oracle.run_f32(d, "average")
    assert ctx.run(torch.from_numpy(junk).cuda(), "average").tobytes() == exp.tobytes()
    out = torch.zeros(149 * 16, dtype=torch.uint8, device="cuda")
    ctx.run(torch.from_numpy(junk).cuda(), "average", out=out)
    ctx.sync()
    assert out.cpu().numpy().tobytes() == exp.tobytes()
    for value in (np.inf, np.nan, 2.0 ** 101):
        bad = d.copy()
        bad[5, 140] = value
        t = torch.from_numpy(bad).cuda()
        rec = np.full(149, 7, np.int32).repeat(4)
        before = rec.tobytes()
        rc = hac.load_library().hac_run(ctx._h, ctypes.c_void_p(t.data_ptr()), 150, 2,
                                        ctypes.c_void_p(rec.ctypes.data), 0, None)
        assert rc == hac.HAC_EINPUT and rec.tobytes() == before
    assert ctx.run(torch.from_numpy(d).cuda(), "average").tobytes() == exp.tobytes()
