"""Small runs whose rounds have few pairs are handed over at once: tied values and
single linkage's last merges, whose rounds cost several merges of the kernel behind.
Rounds are counted; records are the oracle's."""
import ctypes
import math

import numpy as np
import pytest

import oracle
import paper_1709_06816_amd as hac
import synth

pytestmark = pytest.mark.gpu


def _chains(n, count):
    """`count` chains that grow by one point a round each, one distance to all before."""
    p = np.random.default_rng(n).permutation(n)
    x = 1.0 + p // count + (p % count) / (2.0 * count)
    near = np.maximum(x[:, None], x[None, :])
    return np.where((p % count)[:, None] == (p % count)[None, :], near, 1e4 + np.abs(x[:, None] - x[None, :])).astype(np.float32)


@pytest.mark.parametrize("n", [256, 301, 512, 1023, 1500])
def test_few_pairs_hand_over_at_once(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    with hac.Context(0) as ctx:
        for name, link, d in (("quantized", "single", synth.quantized_matrix(n, n, levels=50)),
                              ("constant", "single", np.full((n, n), 1.5, np.float32)),
                              ("chains", "complete", _chains(n, 2)), ("chains", "single", _chains(n, 2)),
                              ("constant", "average", np.full((n, n), 1.5, np.float32))):
            got = ctx.run(torch.from_numpy(np.ascontiguousarray(d)).cuda(), link)
            st = ctx.stats()
            rounds, over = ctypes.c_int32(), ctypes.c_int32()
            hac.load_library().hac_internal_ordered_rounds(ctx._h, ctypes.byref(rounds), ctypes.byref(over))
            rounds, over = (rounds.value, over.value) if link == "average" else (st["rounds"], st["handed_over"])
            print("hand-over: %s n=%d %s after %d rounds" % (name, n, link, rounds), flush=True)
            assert got.tobytes() == oracle.run_f32(d, link).tobytes()
            # Ordered rounds of one tied merge in every second exchange: the running mean
            # (1/256, a sixteenth new each time) falls from what clustered points make
            # to below two merges, rounding and the alternation within 32 units.
            start = 256 * min(16.0, max(3.0, 0.2 * n ** 0.5))
            most = math.ceil(math.log(352.0 / (start - 128.0)) / math.log(15.0 / 16.0)) + 2
            assert over == 1 and rounds <= (most if link == "average" else 4)


@pytest.mark.parametrize("n", [208, 260, 400])
def test_last_merges_of_single_linkage(n):
    """Uniform values: single linkage is one growing cluster soon, a merge a round."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    d = synth.uniform_matrix(n, n)
    with hac.Context(0) as ctx:
        got = ctx.run(torch.from_numpy(d).cuda(), "single")
        st = ctx.stats()
    print("hand-over: uniform n=%d after %d rounds" % (n, st["rounds"]), flush=True)
    assert got.tobytes() == oracle.run_f32(d, "single").tobytes()
    assert st["handed_over"] == 1 and st["rounds"] < n // 5
