"""Calls that wait for their counters, on a capturing stream: they fail, record
nothing, and leave the handle as it was (what comes after equals the same calls
on a handle that saw no capture)."""
import numpy as np
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


def test_extract_on_a_capturing_stream():
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    dims = (72, 50, 41)
    f = fields.turbulence_torch(*dims, seed=31, n_modes=64, kmax=1.0 / 16)
    words = bc.encode(f, 8)
    isos = [float(x) for x in np.linspace(-0.6, 0.6, 4, dtype=np.float32)]
    vol, ref = (bc.Volume(words, dims, "f32", 8) for _ in range(2))
    blocks = bc.blocks_from_field(f)
    fv, fref = bc.FieldVolume(blocks, dims), bc.FieldVolume(blocks, dims)
    dense = bc.DenseMC(dims)
    batch = bc.Batch([ref], [(0, iso) for iso in isos])
    soups = batch.run()[0].clone()
    out = torch.empty((1 << 20, 4), dtype=torch.int32, device="cuda")

    def same(a, b, iso):
        rc, T = a.extract_into(iso, out)
        want, T_ref = b.extract(iso)
        assert rc == 0 and T == T_ref > 0 and torch.equal(out[: 3 * T], want)
        return T

    same(vol, ref, isos[0])
    T = same(fv, fref, isos[0])
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    say("[capture] calls on a capturing stream")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        x += 1
        assert vol.extract_into(isos[1], out)[0] == bc._capi.E_HIP
        assert fv.extract_into(isos[1], out)[0] == bc._capi.E_HIP
        with pytest.raises(bc.BcmcError):
            dense.extract_into(f, isos[1], out)
        assert batch.run_into(out)[0] == bc._capi.E_HIP
    for _ in range(3):   # the capture holds the caller's own work alone
        graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 3).all())
    gV = torch.randn(3 * T, 3, device="cuda")
    (a, ai), (b, bi) = fv.backward(isos[0], gV), fref.backward(isos[0], gV)
    # float atomics: two runs differ by the order of a sample's few sums
    assert torch.allclose(a, b, rtol=1e-5, atol=1e-5 * float(b.abs().max())) and torch.equal(ai, bi)
    for iso in isos[1:] + isos[:1]:
        same(vol, ref, iso)
        same(fv, fref, iso)
    for got, want in zip(vol.cache_state(), ref.cache_state()):
        assert np.array_equal(got, want)
    rc, T = dense.extract_into(f, isos[1], out)
    assert rc == 0 and T == fref.extract(isos[1])[1]
    assert torch.equal(batch.run()[0], soups)
    info = batch.info()
    assert info["n_new"] == 0 and info["graph"] == 1   # the store and the graph are kept
    for h in (batch, vol, ref, fv, fref, dense):
        h.close()
