"""The batch's lists where a volume has more units than one total covers: one
group of units to the last one, and volumes of two and three groups beside small
ones; cold, resident and partly resident, each job's slice against a single extract
of its volume."""
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims_list", [
    [(36, 20, 12), (256, 256, 512), (40, 40, 41)],       # 512 units
    [(512, 256, 260), (36, 20, 12), (384, 512, 384)],    # 520 units; 1152
])
def test_batch_groups(dims_list):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    vols = []
    for v, d in enumerate(dims_list):
        f = fields.turbulence_torch(*d, seed=580 + v, n_modes=24, kmax=1.0 / 24)
        vols.append(bc.Volume(bc.encode(f, 4), d, "f32", 4))
    jobs = [(v, iso) for iso in (0.25, -0.5) for v in (1, 0, 2)]
    say(f"[batch groups] {[x.n_blocks for x in vols]} blocks, {len(jobs)} jobs")
    ref = []
    for v, iso in jobs:
        verts, T = vols[v].extract(iso)
        assert T > 0
        ref.append(verts.clone())
    batch = bc.Batch(vols, jobs)

    def check():
        verts, offs = batch.run()
        for j, r in enumerate(ref):
            assert torch.equal(verts[int(offs[j]): int(offs[j + 1])], r), j

    check()                                                                 # cold
    check()                                                                 # resident
    batch.reset()
    batch.set_isos([i if k < 3 else 99.0 for k, (_, i) in enumerate(jobs)])
    batch.run()
    batch.set_isos([i for _, i in jobs])
    check()                                                                 # partly resident
    batch.close()
    for v in vols:
        v.close()
