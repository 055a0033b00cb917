"""The in-place round engine at small sizes (by default it runs above n = 32768, and
behind the contraction engine): byte-identical merge lists to the CPU oracle on tied
and untied input, any number of workgroups, more pairs than one round takes, the
hand-over, rejected input and its bounded waits."""
import time

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
        assert hac.load_library().hac_internal_rounds_in_place(c._h, 1) == hac.HAC_OK
        c.set_option(hac.OPT_TIMEOUT_MS, 20000)
        yield c


def _run(ctx, d, link, rounds=2, wgs=0):
    import torch
    ctx.set_option(hac.OPT_ROUNDS, rounds)
    ctx.set_option(hac.OPT_WORKGROUPS, wgs)
    try:
        got = ctx.run(torch.from_numpy(np.ascontiguousarray(d)).cuda(), link)
        return got, ctx.stats()
    finally:
        ctx.set_option(hac.OPT_ROUNDS, 1)
        ctx.set_option(hac.OPT_WORKGROUPS, 0)


CASES = [
    ("mixture", lambda n: synth.mixture_8192(seed=n, n=n)),
    ("rmsd_like", lambda n: synth.rmsd_like(seed=n, n=n)),
    ("quantized", lambda n: synth.quantized_matrix(n, n, levels=3)),
    ("constant", lambda n: np.full((n, n), 2.5, np.float32)),
    ("negative", lambda n: synth.uniform_matrix(n, n, -1.0, 1.0)),
    ("lattice", lambda n: synth.euclidean_matrix(np.random.default_rng(n).integers(0, 4, size=(n, 2)).astype(float))),
]


@pytest.mark.parametrize("link", ["single", "complete"])
@pytest.mark.parametrize("name,gen", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("n", [2, 3, 64, 65, 131, 700])
def test_in_place_matches_oracle(ctx, link, name, gen, n):
    d = gen(n)
    print("in place: %s n=%d %s" % (name, n, link), flush=True)
    got, st = _run(ctx, d, link)
    assert got.tobytes() == oracle.run_f32(d, link).tobytes()
    assert st["rounds"] >= 1 and st["handed_over"] == 0


@pytest.mark.parametrize("wgs", [1, 2, 7, 33])
@pytest.mark.parametrize("link", ["single", "complete"])
def test_in_place_any_workgroup_count(ctx, link, wgs):
    d = synth.rmsd_like(seed=77, n=1501)
    print("in place: rmsd_like n=1501 %s on %d workgroups" % (link, wgs), flush=True)
    got, st = _run(ctx, d, link, wgs=wgs)
    assert st["workgroups"] == wgs
    assert got.tobytes() == oracle.run_f32(d, link).tobytes()


@pytest.mark.parametrize("link", ["single", "complete"])
def test_in_place_more_pairs_than_one_round_takes(ctx, link):
    rng = np.random.default_rng(5)
    pts = np.repeat(rng.uniform(-100.0, 100.0, size=(2500, 16)), 2, axis=0) + rng.normal(0.0, 0.01, size=(5000, 16))
    d = synth.euclidean_matrix(pts)
    print("in place: 2500 tight pairs %s" % link, flush=True)
    got, _ = _run(ctx, d, link)
    assert got.tobytes() == oracle.run_f32(d, link).tobytes()


@pytest.mark.parametrize("link", ["single", "complete"])
def test_in_place_hands_over(ctx, link):
    for name, d in (("quantized", synth.quantized_matrix(2000, seed=31, levels=6)),
                    ("quantized", synth.quantized_matrix(1200, seed=34, levels=4)),
                    ("rmsd_like", synth.rmsd_like(seed=33, n=3000))):
        for wgs in (0, 5):
            print("in place: automatic %s %s n=%d wgs=%d" % (link, name, len(d), wgs), flush=True)
            got, st = _run(ctx, d, link, rounds=1, wgs=wgs)
            assert st["handed_over"] == 1
            assert got.tobytes() == oracle.run_f32(d, link).tobytes()


def test_in_place_rejects_and_times_out(ctx):
    import torch
    d = synth.mixture_8192(seed=91, n=3000)
    exp = oracle.run_f32(d, "complete").tobytes()
    bad = d.copy()
    bad[3, 900] = np.nan
    with pytest.raises(hac.HacError) as e:
        ctx.run(torch.from_numpy(bad).cuda(), "single")
    assert e.value.code == hac.HAC_EINPUT
    t = torch.from_numpy(d).cuda()
    ctx.set_option(hac.OPT_TIMEOUT_MS, 100)
    ctx.set_option(hac.OPT_INJECT_STALL, 1)
    try:
        print("in place: stalled exchange", flush=True)
        t0 = time.perf_counter()
        with pytest.raises(hac.HacError) as e:
            ctx.run(t, "complete", preserve=True)
        assert e.value.code == hac.HAC_ETIMEDOUT and time.perf_counter() - t0 < 10.0
    finally:
        ctx.set_option(hac.OPT_INJECT_STALL, 0)
        ctx.set_option(hac.OPT_TIMEOUT_MS, 20000)
    assert ctx.run(t, "complete", preserve=True).tobytes() == exp
