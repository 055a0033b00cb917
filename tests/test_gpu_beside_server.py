"""Small calls beside a busy server: the serving kernel holds all but a few compute
units for as long as it has jobs, and only launches of a few plain workgroups get
through beside it.  Calls of up to 256 items are made of such launches then: they
complete while the server is busy, with the oracle's records."""
import time

import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu

CALLS = [("complete", 100), ("complete", 145), ("complete", 256), ("single", 200), ("single", 256), ("average", 193),
         ("average", 256), ("weighted", 224), ("ward", 256), ("centroid", 256)]


@pytest.mark.parametrize("same_context", [True, False])
def test_small_calls_complete_beside_a_busy_server(same_context):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    mats = [synth.mixture_8192(seed=n, n=n) for _, n in CALLS]
    exps = [oracle.run_f32(d, link).tobytes() for d, (link, _) in zip(mats, CALLS)]
    devs = [torch.from_numpy(d).cuda() for d in mats]
    big = torch.from_numpy(synth.batch_instance(6000, 1)).pin_memory()
    with hac.Context(0) as ctx, hac.Context(0) as other:
        run = ctx if same_context else other
        for d, (link, _) in zip(reversed(devs), reversed(CALLS)):  # largest first: the workspace is there
            run.run(d, link, preserve=True)
        with hac.Server(ctx, budget_bytes=1 << 30, max_jobs=256, max_n=6000) as srv:
            run.set_option(hac.OPT_TIMEOUT_MS, 500)
            tickets = [srv.submit(big, "average") for _ in range(200)]
            while srv.stats()["completed"] == 0:
                time.sleep(0.001)
            for d, exp, (link, n) in zip(devs, exps, CALLS):
                print("beside a server: %s n=%d" % (link, n), flush=True)
                t0 = time.perf_counter()
                got = run.run(d, link, preserve=True)
                took, st = time.perf_counter() - t0, srv.stats()
                print("  %.1f ms on %d workgroups; %d jobs left" % (took * 1e3, run.stats()["workgroups"],
                                                                    200 - st["completed"]), flush=True)
                assert got.tobytes() == exp
                assert st["completed"] < 150, "the server is running out of jobs: nothing shown"
            while srv.stats()["completed"] < 200:
                time.sleep(0.01)
            exp = oracle.run_f32(synth.batch_instance(6000, 1), "average").tobytes()
            assert all(srv.poll(t).tobytes() == exp for t in tickets)
