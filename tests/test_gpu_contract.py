"""GPU tests of the contraction engine (single and complete linkage by rounds on
a shrinking matrix): byte-identical merge lists to the CPU oracle where the
threads per row change, on row lengths of every alignment, with retired columns
kept in place (single linkage, few pairs per round) and handed back to their
slots, and at the largest size it takes, beside the in-place engine above it."""
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
        c.set_option(hac.OPT_TIMEOUT_MS, 20000)
        yield c


def _run(ctx, d, link, rounds, wgs=0):
    import torch
    ctx.set_option(hac.OPT_ROUNDS, rounds)
    ctx.set_option(hac.OPT_WORKGROUPS, wgs)
    try:
        got = ctx.run(torch.from_numpy(np.ascontiguousarray(d)).cuda(), link)
        return got, ctx.stats()
    finally:
        ctx.set_option(hac.OPT_ROUNDS, 1)
        ctx.set_option(hac.OPT_WORKGROUPS, 0)


@pytest.mark.parametrize("link", ["single", "complete"])
@pytest.mark.parametrize("n", [4, 63, 67, 255, 513, 1026, 2051, 2300])
def test_contract_matches_oracle(ctx, link, n):
    for name, d in (("mixture", synth.mixture_8192(seed=n, n=n)), ("rmsd_like", synth.rmsd_like(seed=n, n=n)),
                    ("negative", synth.uniform_matrix(n, n, -1.0, 1.0)),
                    ("subnormal", synth.uniform_matrix(n, n) * np.float32(1e-38))):
        exp = oracle.run_f32(d, link).tobytes()
        for rounds, wgs in ((1, 0), (2, 0), (2, 3)):
            print("contract: %s n=%d %s rounds=%d wgs=%d" % (name, n, link, rounds, wgs), flush=True)
            got, st = _run(ctx, d, link, rounds, wgs)
            assert got.tobytes() == exp
            assert st["rounds"] > 0 or rounds == 1


def test_contract_chains_in_place(ctx):
    """Points on a line with growing gaps beside scattered ones: single linkage
    grows chains, so most rounds have few pairs and update in place."""
    rng = np.random.default_rng(3)
    line = np.cumsum(1.0 + 1e-4 * np.arange(1200))[:, None] * np.array([[1.0, 0.0, 0.0]])
    pts = np.concatenate([line, rng.normal(0, 200.0, size=(800, 3))])
    d = synth.euclidean_matrix(pts[rng.permutation(len(pts))])
    exp = oracle.run_f32(d, "single").tobytes()
    for rounds in (1, 2):
        got, st = _run(ctx, d, "single", rounds)
        assert got.tobytes() == exp


def test_largest_size_and_the_engine_above(ctx):
    """n = 32768 (the last the contraction engine takes) and 32769, 32771 (in
    place) against one merge per step."""
    import torch
    for n, link in ((32768, "complete"), (32769, "complete"), (32771, "single")):
        d = torch.empty((n, n), dtype=torch.float32, device="cuda")
        x = torch.from_numpy(synth.gaussian_mixture(np.random.default_rng(n), n, 8, 32, 0.5, 2.0).astype(np.float32))
        x = x.cuda()
        for a in range(0, n, 4096):
            d[a:a + 4096] = (x[a:a + 4096, None, :] - x[None, :, :]).square().sum(-1).sqrt()
        print("contract: n=%d %s" % (n, link), flush=True)
        got = ctx.run(d, link, preserve=True)
        assert ctx.stats()["rounds"] > 0
        ctx.set_option(hac.OPT_ROUNDS, 0)
        exp = ctx.run(d, link)
        ctx.set_option(hac.OPT_ROUNDS, 1)
        assert got.tobytes() == exp.tobytes()
