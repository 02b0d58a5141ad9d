"""A cache budget that no memory holds: the call fails, extracts then report the
cap, and the next budget that fits gives the same soup."""
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


def test_budget_that_does_not_fit():
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    dims = (72, 50, 41)
    f = fields.turbulence_torch(*dims, seed=32, n_modes=64, kmax=1.0 / 16)
    vol = bc.Volume(bc.encode(f, 8), dims, "f32", 8)
    want, T = vol.extract(0.1)
    want = want.clone()
    out = torch.empty((3 * T, 4), dtype=torch.int32, device="cuda")
    slots = 2 * torch.cuda.get_device_properties(0).total_memory // 256
    say(f"[budget] {slots} slots, twice the device's memory")
    with pytest.raises(bc.BcmcError):
        vol.set_cache_budget(0, 256 * min(slots, 2 ** 31 - 2))
    for _ in range(2):
        assert vol.extract_into(0.1, out)[0] == bc._capi.E_CACHE_CAP
        vol.reset_cache()
    assert len(vol.cache_state()[1]) == 0
    vol.set_cache_budget(0, 0)
    rc, got = vol.extract_into(0.1, out)
    assert rc == 0 and got == T and torch.equal(out, want)
    vol.close()
