"""The batch's flags and lists where their units of 1024 blocks end: volumes of
1 block, 1023, 1024, 1025 and several units, more jobs of a volume than are
counted between two barriers, jobs in mixed order, partly resident stores; each
job's slice against a single extract of its volume."""
import numpy as np
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims_list,jobs_per_vol", [
    ([(4, 4, 4), (64, 64, 16)], 3),
    ([(132, 44, 12), (64, 64, 16), (5, 20, 820), (3, 2, 2)], 2),   # 1089, 1024, 2050 and 1 blocks
    ([(92, 44, 16), (40, 40, 41)], 37),                             # 1012 and 1100 blocks, 37 jobs each
])
def test_batch_units(dims_list, jobs_per_vol):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    vols, jobs = [], []
    rng = np.random.default_rng(97)
    for v, d in enumerate(dims_list):
        f = fields.turbulence_torch(*d, seed=970 + v, n_modes=32, kmax=1.0 / 16)
        vols.append(bc.Volume(bc.encode(f, 8), d, "f32", 8))
        jobs += [(v, float(np.float32(x))) for x in rng.uniform(-1.6, 1.6, jobs_per_vol)]
    rng.shuffle(jobs)
    jobs = [(int(v), float(i)) for v, i in jobs]
    say(f"[batch units] {[x.n_blocks for x in vols]} blocks, {len(jobs)} jobs")
    ref = []
    for v, iso in jobs:
        verts, T = vols[v].extract(iso)
        ref.append(verts.clone())
    batch = bc.Batch(vols, jobs)

    def check(isos_changed=False):
        verts, offs = batch.run()
        for j, r in enumerate(ref):
            assert torch.equal(verts[int(offs[j]): int(offs[j + 1])], r), j

    check()                                     # cold
    check()                                     # everything resident
    batch.reset()
    batch.set_isos([i if k % 2 else 99.0 for k, (_, i) in enumerate(jobs)])   # half the jobs, a part resident
    batch.run()
    batch.set_isos([i for _, i in jobs])
    check()
    assert batch.info()["n_resident"] == len(set().union(*_used(vols, jobs)))
    batch.close()
    for v in vols:
        v.close()


def _used(vols, jobs):
    """(volume, block) of every block active for some job."""
    import torch
    out = torch.empty((1, 4), dtype=torch.int32, device="cuda")
    for v, iso in jobs:
        vols[v].extract_into(iso, out)
        yield {(v, int(b)) for b in vols[v].active()[1]}
