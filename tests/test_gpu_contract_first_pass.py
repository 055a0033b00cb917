"""The contraction engine's first pass (every row's minimum, one barrier per row)
where a row takes several waves and a workgroup several rows one after the other:
128 to 1024 threads a row, many rows per workgroup, tied values, against the
one-merge-per-step kernel on the same matrix."""
import pytest

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


@pytest.mark.parametrize("link", ["single", "complete"])
@pytest.mark.parametrize("n,wgs", [(2049, 0), (2049, 1), (4099, 2), (8200, 0), (8193, 5), (16501, 0)])
def test_rows_of_several_waves(ctx, link, n, wgs):
    import torch
    d = torch.from_numpy(synth.rmsd_like(seed=n, n=n)).cuda()
    print("contract, first pass: n=%d %s workgroups=%d" % (n, link, wgs), flush=True)
    ctx.set_option(hac.OPT_WORKGROUPS, wgs)
    try:
        got = [ctx.run(d, link, preserve=True).tobytes() for _ in range(2)]
        assert ctx.stats()["rounds"] > 0
        ctx.set_option(hac.OPT_ROUNDS, 0)
        exp = ctx.run(d, link, preserve=True).tobytes()
    finally:
        ctx.set_option(hac.OPT_ROUNDS, 1)
        ctx.set_option(hac.OPT_WORKGROUPS, 0)
    assert got == [exp, exp]
