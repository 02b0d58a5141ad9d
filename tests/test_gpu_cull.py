"""Active blocks, may-emit flags and the block lists against the oracle over
the forms of the cull and the compaction: one workgroup per tile and the
queue of live tiles, rows of blocks that cross rounds of 4096, tiles live in
one call and dead in the next, and flags that new ranges make meaningless."""
import numpy as np
import pytest

from synthetic import fields
from tests.gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu


def _hull_2x2x2(rg, nb3):
    """(lo, hi) over each block and its positive neighbours, [N_b] each."""
    nbx, nby, nbz = nb3
    out = []
    for k, op in ((0, np.minimum), (1, np.maximum)):
        v = np.pad(rg[:, k].reshape(nbz, nby, nbx), ((0, 1),) * 3, mode="edge")
        for axis in range(3):
            a = [slice(None)] * 3
            b = [slice(None)] * 3
            a[axis], b[axis] = slice(0, -1), slice(1, None)
            v = op(v[tuple(a)], v[tuple(b)])
        out.append(v.ravel())
    return out


def _check(orc, vol, dims, iso):
    rg = vol.ranges()
    act, ids, emit = vol.active(with_flags=True)
    want = orc.active_blocks(rg, dims, iso)
    assert np.array_equal(act, want)
    assert np.array_equal(ids, np.flatnonzero(want))
    lo, hi = _hull_2x2x2(rg, orc.block_dims(*dims))
    may = (lo < np.float32(iso)) & (np.float32(iso) <= hi)
    assert np.array_equal(emit.astype(bool), may)
    assert vol.stats()["n_candidates"] == int(may.sum())


@pytest.mark.parametrize("dims", [(133, 70, 51),        # 34 blocks a row: 2 tiles, rows across rounds
                                  (4, 300, 290),        # 1 block a row
                                  (5, 2080, 2075)])     # 4225 tiles: queued
def test_cull_matches_oracle(orc, dims):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    f = fields.turbulence_torch(*dims, seed=81, n_modes=32, kmax=1.0 / 32)
    out = torch.empty((16, 4), dtype=torch.int32, device="cuda")
    vol = bc.Volume(bc.encode(f, 4), dims, "f32", 4)
    isos = [float(np.float32(x)) for x in (0.0, 1.5, -1.5, 1.5, 9.0, 0.3)]
    say(f"[cull] {dims}: {vol.n_blocks} blocks")
    for iso in isos:
        vol.extract_into(iso, out)
        _check(orc, vol, dims, iso)
    blocks = vol.decode_all()                # the ranges are formed anew
    vol.extract_into(isos[1], out)
    _check(orc, vol, dims, isos[1])
    fv = bc.FieldVolume(blocks, dims)
    fv.extract_into(isos[0], out)
    fv.rebind((blocks + 0.7).contiguous())   # other ranges under the same flags
    fv.extract_into(isos[0], out)
    _check(orc, fv, dims, isos[0])
    vol.close()
    fv.close()
