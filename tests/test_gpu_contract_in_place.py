"""Complete linkage whose rounds have few pairs: the contraction engine, which
streams the whole matrix in a round, leaves the run to the in-place round engine
queued behind it, which resumes from its live clusters, sizes and records (and may
hand over in turn to the one-merge-per-step kernel).  Against that kernel alone."""
import pytest

import paper_1709_06816_amd as hac

pytestmark = pytest.mark.gpu


def _lines(torch, n, count, tied):
    """`count` rows of points that grow one pair a round each: on lines with growing
    gaps, or (tied) with one distance from a point to all before it."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + count)
    p = torch.randperm(n, generator=gen, device="cuda")
    line, k = (p % count).double(), torch.div(p, count, rounding_mode="floor").double()
    x = 1.0 + k + line / (2 * count) if tied else k + k * k * (0.5 / 1024) + k * line * 1e-5
    d = torch.empty((n, n), dtype=torch.float32, device="cuda")
    for a in range(0, n, 2048):
        r = slice(a, a + 2048)
        near = torch.maximum(x[r, None], x[None, :]) if tied else (x[r, None] - x[None, :]).abs()
        far = 1e6 + 100.0 * (line[r, None] - line[None, :]).abs() + 0.01 * (x[r, None] - x[None, :]).abs()
        d[r] = torch.where(line[r, None] == line[None, :], near, far).float()
    return d


@pytest.mark.parametrize("n,count,tied", [(8193, 2, False), (8500, 4, False), (12001, 16, False), (12000, 16, True),
                                          (32768, 16, False)])
def test_few_pairs_go_on_in_place(n, count, tied):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    d = _lines(torch, n, count, tied)
    with hac.Context(0) as ctx:
        ctx.set_option(hac.OPT_TIMEOUT_MS, 20000)
        ctx.set_option(hac.OPT_ROUNDS, 0)
        exp = ctx.run(d, "complete", preserve=True).tobytes()
        for rounds, wgs in ((1, 0), (2, 0), (2, 40)):
            if wgs and n > 20000:
                continue
            ctx.set_option(hac.OPT_ROUNDS, rounds)
            ctx.set_option(hac.OPT_WORKGROUPS, wgs)
            print("contract, in place: n=%d lines=%d tied=%d rounds=%d workgroups=%d" % (n, count, tied, rounds, wgs),
                  flush=True)
            got = ctx.run(d, "complete", preserve=True)
            st = ctx.stats()
            assert got.tobytes() == exp
            # A run streamed in every round moves two thirds of rounds * n^2 entries;
            # untied lines rescan a few rows a round in place.
            if rounds == 2 and not tied:
                assert st["rounds"] > n // (4 * count) and st["rounds_rescan_elems"] < st["rounds"] * n * n // 4, st


def test_many_pairs_stay():
    """Clustered points: every round has pairs enough, nothing is left to the engine
    behind (which would rescan rows, not stream matrices)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import synth
    n = 10000
    d = torch.from_numpy(synth.rmsd_like(seed=5, n=n)).cuda()
    with hac.Context(0) as ctx:
        got = ctx.run(d, "complete", preserve=True)
        st = ctx.stats()
        ctx.set_option(hac.OPT_ROUNDS, 0)
        assert got.tobytes() == ctx.run(d, "complete", preserve=True).tobytes()
    print("contract: n=%d, %d rounds" % (n, st["rounds"]), flush=True)
    assert st["handed_over"] == 0 and st["rounds"] < 200
