"""Served jobs on as many workgroups as the server has to spare: sizes around the
rule's steps, alone (workgroups to spare) and in a burst of more members than
workgroups (the first jobs on larger groups than the last), each with the oracle's
records."""
import time

import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,count", [((512, 513, 1023, 1024), 4), ((1024, 1025, 640, 2049), 200)])
def test_groups_by_load(sizes, count):
    import torch
    import paper_1709_06816_amd as hac
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mats = [synth.batch_instance(n, 900 + n) for n in sizes]
    exps = [[oracle.run_f32(m, link).tobytes() for link in range(4)] for m in mats]
    pinned = [torch.from_numpy(m).pin_memory() for m in mats]
    with hac.Context(0) as ctx, hac.Server(ctx, budget_bytes=4 << 30, max_jobs=256, max_n=2304) as srv:
        for wave in range(2):
            jobs = [(k % len(sizes), (k // len(sizes) + wave) % 4) for k in range(count)]
            print("[gpu-serve-groups] %d jobs of %s, wave %d" % (count, sizes, wave), flush=True)
            tickets = [srv.submit(pinned[m], link) for m, link in jobs]
            for t, (m, link) in zip(tickets, jobs):
                got = srv.poll(t)
                while got is None:
                    time.sleep(0.0005)
                    got = srv.poll(t)
                assert got.tobytes() == exps[m][link], (sizes[m], link)
