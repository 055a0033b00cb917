"""Single linkage on tied values in the contraction engine, rounds to the end:
rounds update in place until a share of the columns have retired, then one
contracts, over and over, so that every contraction starts from a mask of retired
columns that the next round must find empty.  Against the CPU oracle."""
import numpy as np
import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu


def _lattice(n):
    return synth.euclidean_matrix(np.random.default_rng(n).integers(0, 9, size=(n, 4)).astype(np.float64))


@pytest.mark.parametrize("n", [1100, 2048, 3001])
@pytest.mark.parametrize("name,gen", [("rmsd_like", lambda n: synth.rmsd_like(seed=n, n=n)),
                                      ("quantized", lambda n: synth.quantized_matrix(n, n, levels=200)),
                                      ("lattice", _lattice)], ids=["rmsd_like", "quantized", "lattice"])
def test_in_place_and_contracted_rounds_in_turn(name, gen, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    d = np.ascontiguousarray(gen(n))
    exp = oracle.run_f32(d, "single").tobytes()
    with hac.Context(0) as ctx:
        ctx.set_option(hac.OPT_TIMEOUT_MS, 20000)
        ctx.set_option(hac.OPT_ROUNDS, 2)
        for wgs in (0, 7):
            ctx.set_option(hac.OPT_WORKGROUPS, wgs)
            print("contract, retired columns: %s n=%d workgroups=%d" % (name, n, wgs), flush=True)
            got = ctx.run(torch.from_numpy(d).cuda(), "single")
            st = ctx.stats()
            assert got.tobytes() == exp
            assert st["rounds"] > 50
            # Contracting in every round streams twice the matrix each time, two
            # thirds of rounds * n^2 over the run; up to m = 1024 the engine does.
            if n > 2048:
                assert st["rounds_rescan_elems"] < 1024 ** 3 + st["rounds"] * n * n // 5, st
