"""GPU tests of the ordered-round engine (group average, weighted average and
Ward linkage, several merges per exchange): byte-identical merge lists to the
CPU oracle at the edges of its column blocks and workgroup counts, on inputs
where rounds shrink to one merge (ties, zeros, negative and subnormal values),
with and without the hand-over, and its bounded waits."""
import numpy as np
import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu

LINKS = ("average", "weighted", "ward")


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
        return ctx.run(torch.from_numpy(np.ascontiguousarray(d)).cuda(), link)
    finally:
        ctx.set_option(hac.OPT_ROUNDS, 1)
        ctx.set_option(hac.OPT_WORKGROUPS, 0)


def _pairs(n, seed):
    """Tight pairs far apart: the first round offers n / 2 merges."""
    rng = np.random.default_rng(seed)
    c = rng.uniform(-100.0, 100.0, size=((n + 1) // 2, 8))
    return synth.euclidean_matrix((np.repeat(c, 2, axis=0) + rng.normal(0, 0.01, size=(2 * len(c), 8)))[:n])


CASES = [
    ("mixture", lambda n: synth.mixture_8192(seed=n, n=n)),
    ("rmsd_like", lambda n: synth.rmsd_like(seed=n, n=n)),
    ("quantized", lambda n: synth.quantized_matrix(n, n, levels=3)),
    ("negative", lambda n: synth.uniform_matrix(n, n, -1.0, 1.0)),
    ("zeros", lambda n: np.where(synth.uniform_matrix(n, n) < 0.5, np.float32(0), synth.uniform_matrix(n, n))),
    ("subnormal", lambda n: synth.uniform_matrix(n, n) * np.float32(1e-38)),
    ("large", lambda n: synth.uniform_matrix(n, n) * np.float32(2.0 ** 99)),
    ("tight pairs", lambda n: _pairs(n, n)),
]


@pytest.mark.parametrize("name,gen", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("n", [2, 3, 64, 65, 257, 700])
def test_order_matches_oracle(ctx, name, gen, n):
    d = gen(n)
    for link in LINKS:
        exp = oracle.run_f32(d, link).tobytes()
        for rounds in (1, 2):
            print("order: %s n=%d %s rounds=%d" % (name, n, link, rounds), flush=True)
            assert _run(ctx, d, link, rounds).tobytes() == exp


@pytest.mark.parametrize("link", LINKS)
@pytest.mark.parametrize("wgs", [2, 3, 5, 10, 20, 40])
def test_order_any_column_block(ctx, link, wgs):
    """1024 down to 64 columns per workgroup, the last block partly filled."""
    d = synth.mixture_8192(seed=3, n=1281)
    print("order: n=1281 %s on at most %d workgroups" % (link, wgs), flush=True)
    assert _run(ctx, d, link, 2, wgs).tobytes() == oracle.run_f32(d, link).tobytes()


def test_order_many_workgroups_match_one_merge_per_step(ctx):
    """Above 128 workgroups one of them selects the merges; above n=32768 the
    cluster sizes are read from memory.  Against the one-merge-per-step
    kernel (the oracle needs hours there)."""
    import torch
    for n, link, wgs in ((8257, "ward", 0), (8257, "average", 64), (33000, "average", 0)):
        d = torch.empty((n, n), dtype=torch.float32, device="cuda")
        x = torch.from_numpy(synth.gaussian_mixture(np.random.default_rng(n), n, 8, 32, 0.5, 2.0).astype(np.float32))
        x = x.cuda()
        for a in range(0, n, 4096):
            d[a:a + 4096] = (x[a:a + 4096, None, :] - x[None, :, :]).square().sum(-1).sqrt()
        print("order: n=%d %s wgs=%d" % (n, link, wgs), flush=True)
        ctx.set_option(hac.OPT_WORKGROUPS, wgs)
        got = ctx.run(d, link, preserve=True)
        ctx.set_option(hac.OPT_WORKGROUPS, 0)
        ctx.set_option(hac.OPT_ROUNDS, 0)
        exp = ctx.run(d, link)
        ctx.set_option(hac.OPT_ROUNDS, 1)
        assert got.tobytes() == exp.tobytes()


def test_order_stall_times_out_and_recovers(ctx):
    import torch
    d = synth.mixture_8192(seed=91, n=3000)
    t = torch.from_numpy(d).cuda()
    ctx.set_option(hac.OPT_TIMEOUT_MS, 100)
    for wgs in (8, 0):
        ctx.set_option(hac.OPT_WORKGROUPS, wgs)
        ctx.set_option(hac.OPT_INJECT_STALL, 1)
        try:
            print("order: stalled exchange wgs=%d" % wgs, flush=True)
            with pytest.raises(hac.HacError) as e:
                ctx.run(t, "average", preserve=True)
            assert e.value.code == hac.HAC_ETIMEDOUT
        finally:
            ctx.set_option(hac.OPT_INJECT_STALL, 0)
    ctx.set_option(hac.OPT_WORKGROUPS, 0)
    ctx.set_option(hac.OPT_TIMEOUT_MS, 20000)
    assert ctx.run(t, "average", preserve=True).tobytes() == oracle.run_f32(d, "average").tobytes()
