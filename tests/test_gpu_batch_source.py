"""hac_batch with its input kept: each instance's set-up reads the caller's matrix
and writes the working one.  Only the strict upper triangle may be read (the rest
holds NaN here), -0.0 counts as 0, the input's bytes stay, an invalid instance is
reported, and every plan gives the in-place call's records."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,group", [(256, 1), (1024, 1), (1024, 4), (0, 0)])
def test_kept_input(block, group):
    import torch
    import paper_1709_06816_amd as hac
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ns = np.array([2100, 2049, 65, 64, 63, 2, 1, 130, 257], np.int64)
    links = [k % 4 for k in range(len(ns))]
    rng = np.random.default_rng(11)
    offs, total = synth.pack_offsets(ns)
    packed = np.full(total, np.nan, np.float32)
    mats = []
    for k, n in enumerate(ns):
        d = np.full((n, n), np.nan, np.float32)
        iu = np.triu_indices(n, 1)
        v = rng.random(len(iu[0]), dtype=np.float32)
        v[rng.random(len(v)) < 0.01] = -0.0
        d[iu] = v
        packed[offs[k]:offs[k] + n * n] = d.ravel()
        mats.append(np.where(np.isnan(d), np.float32(0), d))
    t = torch.from_numpy(packed).cuda()
    with hac.Context(0) as ctx:
        ctx.set_option(hac.OPT_BATCH_BLOCK, block)
        ctx.set_option(hac.OPT_BATCH_GROUP, group)
        print("[gpu-batch-source] block=%d group=%d" % (block, group), flush=True)
        kept = ctx.batch(t, offs, ns, links, preserve=True)
        assert t.cpu().numpy().tobytes() == packed.tobytes()
        again = ctx.batch(t, offs, ns, links, preserve=True)
        placed = ctx.batch(t.clone(), offs, ns, links)
        assert kept.tobytes() == again.tobytes() == placed.tobytes()
        moff, _ = synth.merge_offsets(ns)
        for k in range(2, len(ns)):
            n = int(ns[k])
            if n > 1:
                assert kept[moff[k]:moff[k] + n - 1].tobytes() == oracle.run_f32(mats[k], links[k]).tobytes(), n
        t[int(offs[4]) + 5] = float("inf")
        with pytest.raises(hac.HacError):
            ctx.batch(t, offs, ns, links, preserve=True)
