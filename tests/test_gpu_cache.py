"""The cache's choice of slots (unused ones first, then the oldest by the
selection over stamps) against the oracle's LRU simulator where the selection
changes its form: more tiles of slots than one workgroup adds up itself, one
and two passes of key digits, and the key base that long runs of calls move."""
import numpy as np
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


def _step(bc, orc, vol, sim, out, dims, rg, iso):
    rc, T = vol.extract_into(float(iso), out)
    assert rc in (0, bc._capi.E_CAPACITY)      # the soup is not looked at
    rc, I_new, ev = sim.update(orc.active_blocks(rg, dims, iso))
    assert rc == 0
    st = vol.stats()
    assert (st["n_new"], st["n_evicted"], st["n_slots"]) == (len(I_new), ev, sim.n_slots)
    for got, want in zip(vol.cache_state(), sim.state()):
        assert np.array_equal(got, want)
    return ev


@pytest.mark.parametrize("dims,init,cap,idle", [
    ((512, 384, 128), 0, 262144, 0),          # 64 tiles: every workgroup adds up the rows
    ((512, 384, 128), 1000, 300000, 0),       # 74 tiles: the rows are scanned
    ((512, 384, 128), 300000, 300000, 5000),  # the same, two digits of keys
    ((40, 37, 33), 0, 500, 3000),             # one tile, two digits
])
def test_evictions_match_simulator(orc, dims, init, cap, idle):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    f = fields.turbulence_torch(*dims, seed=71, n_modes=64, kmax=1.0 / 48)
    vol = bc.Volume(bc.encode(f, 2), dims, "f32", 2)
    vol.set_cache_budget(init * 256, cap * 256)
    rg = vol.ranges()
    out = torch.empty((16, 4), dtype=torch.int32, device="cuda")
    sim = orc.LRU(vol.n_blocks, init, cap)
    isos = [float(np.quantile(rg.mean(1), q)) for q in (0.1, 0.5, 0.9, 0.3, 0.1, 0.7, 0.5)]
    say(f"[cache] {dims}: {vol.n_blocks} blocks, {cap} slots, {idle} idle calls")
    ev = sum(_step(bc, orc, vol, sim, out, dims, rg, i) for i in isos)
    if idle:
        vol.age_cache(idle)
        sim.idle(idle)
        ev += sum(_step(bc, orc, vol, sim, out, dims, rg, i) for i in isos[:4])
    assert ev > 0
    # emptied: every slot unused again
    vol.reset_cache()
    I_slot, S_block, S_age = vol.cache_state()
    assert (I_slot == -1).all() and (S_block[:init] == -1).all() and (S_age[:init] == 1 << 31).all()
    sim = orc.LRU(vol.n_blocks, init, cap)
    for i in isos[:2]:
        _step(bc, orc, vol, sim, out, dims, rg, i)
    vol.close()


def test_key_base_moves_with_repeated_calls(orc):
    """2100 calls of one surface (every used slot stamped each time, then a
    part of them never again), and evictions after them."""
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    dims = (40, 37, 33)
    f = fields.turbulence_torch(*dims, seed=72, n_modes=64, kmax=1.0 / 48)
    vol = bc.Volume(bc.encode(f, 4), dims, "f32", 4)
    vol.set_cache_budget(0, 460 * 256)
    rg = vol.ranges()
    out = torch.empty((16, 4), dtype=torch.int32, device="cuda")
    sim = orc.LRU(vol.n_blocks, 0, 460)
    a, b, c, d = (float(np.quantile(rg.mean(1), q)) for q in (0.1, 0.5, 0.9, 0.3))
    act = orc.active_blocks(rg, dims, b)
    ev = 0
    for first in (a, c):
        ev += _step(bc, orc, vol, sim, out, dims, rg, first)
        for _ in range(1050):
            vol.extract_into(b, out)
            assert sim.update(act)[0] == 0
        ev += sum(_step(bc, orc, vol, sim, out, dims, rg, i) for i in (d, c, a, b))
    assert ev > 0
    vol.close()
