"""The backward's output buffers: written in full whatever they held, at any
4-byte alignment, and nothing beside them.  Tolerance: float32 sums in another
order (the field's gradient adds by atomics)."""
import ctypes as C

import numpy as np
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_gradient_buffers(orc, offset):
    torch = torch_cuda()
    import paper_2009_03254_amd as bcmc
    n = 41   # partial blocks, a buffer of no whole number of workgroups' stores
    say(f"[backward buffers] offset {offset}")
    f = fields.gaussian_blobs(n, 6, seed=31)
    dims = (n, n, n)
    B = orc.field_to_blocks(f)
    iso = float(fields.percentile_iso(f, 60))
    vol = bcmc.FieldVolume(torch.from_numpy(B).cuda(), dims)
    _, T = vol.extract(iso)
    gV = torch.randn((3 * T, 3), generator=torch.Generator().manual_seed(5), dtype=torch.float32).cuda()
    buf = torch.full((B.size + 8,), float("nan"), dtype=torch.float32, device="cuda")
    diso = torch.full((3,), float("nan"), dtype=torch.float32, device="cuda")
    for _ in range(2):
        rc = bcmc.lib().bcmc_backward(vol._h, C.c_float(iso), C.c_void_p(gV.data_ptr()), 3 * T,
                                      C.c_void_p(buf.data_ptr() + 4 * offset), C.c_void_p(diso.data_ptr() + 4),
                                      C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
    vol.close()
    got, di = buf.cpu().numpy(), diso.cpu().numpy()
    want, dio = orc.mc_backward(B, dims, iso, gV.cpu().numpy().astype(np.float64))
    assert np.linalg.norm(got[offset: offset + B.size].astype(np.float64) - want.ravel()) <= 1e-4 * np.linalg.norm(want)
    assert np.isnan(got[:offset]).all() and np.isnan(got[offset + B.size:]).all()
    assert di[1] == pytest.approx(dio, rel=1e-4) and np.isnan(di[0]) and np.isnan(di[2])
