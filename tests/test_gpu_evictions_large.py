"""The cache's evictions against the oracle's LRU simulator where the selection's
first pass is not counted by the compaction (volumes of more than 2048 rounds of
4096 blocks, culled from the queue), and where the rows of one pass are scanned; with
calls enough between for the key base to be looked for again and for two digits."""
import numpy as np
import pytest

from tests.gpu_common import say, torch_cuda
from tests.test_gpu_cache import _step

pytestmark = pytest.mark.gpu


def _sheets(torch, dims):
    """A wavy ramp along z: one sheet per isovalue."""
    x, y, z = (torch.arange(n, device="cuda", dtype=torch.float32) for n in dims)
    plane = 0.3 * torch.sin(0.02 * x)[None, :] * torch.cos(0.017 * y)[:, None]
    return (z * (4.0 / dims[2]) - 2.0)[:, None, None] + plane[None]


@pytest.mark.parametrize("dims,init,cap,idles", [
    ((816, 820, 824), 0, 300000, (200, 600, 5000)),   # 2104 rounds; 8 key bits (scanned, one pass), then two digits
    ((512, 384, 400), 1000, 131072, (300,)),          # 300 rounds, 128 tiles x 512 digits: scanned, one pass
])
def test_evictions_match_simulator_large(orc, dims, init, cap, idles):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    vol = bc.Volume(bc.encode(_sheets(torch, dims), 2), dims, "f32", 2)
    vol.set_cache_budget(init * 256, cap * 256)
    rg = vol.ranges()
    out = torch.empty((16, 4), dtype=torch.int32, device="cuda")
    sim = orc.LRU(vol.n_blocks, init, cap)
    say(f"[cache] {dims}: {vol.n_blocks} blocks, {cap} slots, idle calls {idles}")
    ev = sum(_step(bc, orc, vol, sim, out, dims, rg, i) for i in (-1.0, 0.0, -1.0))
    for idle in idles:
        vol.age_cache(idle)
        sim.idle(idle)
        got = sum(_step(bc, orc, vol, sim, out, dims, rg, i) for i in (1.0, 0.05, -1.0))
        say(f"  after {idle}: {got} evicted, {vol.stats()['n_active']} active")
        ev += got
        assert got > 0
    vol.close()
