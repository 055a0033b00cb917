"""The ordered-round engine is what runs: its exchanges per run on clustered points
are a fraction of the merges, on tied input it hands over (unless told to make every
merge), and sizes and linkages that are not its own leave it alone."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu


def _rounds(ctx):
    r, h = ctypes.c_int32(-1), ctypes.c_int32(-1)
    assert hac.load_library().hac_internal_ordered_rounds(ctx._h, ctypes.byref(r), ctypes.byref(h)) == hac.HAC_OK
    return r.value, h.value


@pytest.mark.parametrize("link", ["average", "weighted", "ward"])
def test_rounds_of_several_merges(link):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    with hac.Context(0) as ctx:
        for name, d, opt, handed in (("mixture", synth.mixture_8192(seed=7, n=2500), 1, 0),
                                     ("constant", np.full((600, 600), 2.5, np.float32), 1, 1),
                                     ("constant", np.full((600, 600), 2.5, np.float32), 2, 0)):
            n = len(d)
            ctx.set_option(hac.OPT_ROUNDS, opt)
            got = ctx.run(torch.from_numpy(d).cuda(), link)
            rounds, over = _rounds(ctx)
            print("order: %s n=%d %s rounds=%d: %d exchanges, handed over %d, %d workgroups" %
                  (name, n, link, opt, rounds, over, ctx.stats()["workgroups"]), flush=True)
            assert got.tobytes() == oracle.run_f32(d, link).tobytes()
            assert over == handed and rounds > 0
            assert ctx.stats()["workgroups"] == (n + 63) // 64
            if name == "mixture":
                assert rounds < n // 4
        ctx.set_option(hac.OPT_ROUNDS, 1)
        for link2, n in (("centroid", 700), ("complete", 700), (link, 150)):
            ctx.run(torch.from_numpy(synth.mixture_8192(seed=7, n=n)).cuda(), link2)
            assert _rounds(ctx) == (0, 0), (link2, n)
