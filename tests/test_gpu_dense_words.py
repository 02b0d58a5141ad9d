"""Dense marching cubes where its words of 64 cells end: rows of 1, 63, 64,
65 and 128 cells, words whose cells are all active (a checkerboard: every cell
four triangles), chunks of one word and of 64, against the oracle's scan."""
import numpy as np
import pytest

from tests.gpu_common import say, to_cuda, torch_cuda

pytestmark = pytest.mark.gpu


def _field(kind, dims, seed):
    nx, ny, nz = dims
    if kind == "noise":
        return np.random.default_rng(seed).standard_normal((nz, ny, nx)).astype(np.float32)
    z, y, x = np.indices((nz, ny, nx))
    if kind == "checker":
        return np.where((x + y + z) % 2, 1.0, -0.75).astype(np.float32)
    return (x * 0.5 + y - 2.0 * z + 0.25).astype(np.float32)   # a plane


@pytest.mark.parametrize("kind", ["noise", "checker", "plane"])
@pytest.mark.parametrize("dims", [(2, 2, 2), (2, 40, 3), (64, 5, 4), (65, 7, 9), (66, 4, 5), (129, 6, 3),
                                  (200, 130, 45)])
def test_dense_words(orc, kind, dims):
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    f = _field(kind, dims, 91)
    say(f"[dense words] {kind} {dims}")
    dm = bc.DenseMC(dims)
    fd = to_cuda(f)
    for iso in (0.0, 0.3):
        v, vb = orc.mc_extract_dense(f, np.float32(iso))
        out = torch.full((len(vb) + 8, 4), -7, dtype=torch.int32, device="cuda")
        rc, T = dm.extract_into(fd, iso, out)
        assert rc == 0 and 3 * T == len(vb)
        got = out.cpu().numpy()
        assert np.array_equal(got[: 3 * T, :3].view(np.uint32), v.view(np.uint32))
        assert np.array_equal(got[: 3 * T, 3].view(np.uint32), vb)
        assert (got[3 * T:] == -7).all()
    dm.close()


@pytest.mark.parametrize("dims", [(512, 120, 120), (512, 512, 128)])
def test_dense_chunks_across_rows(orc, dims):
    """Rows whole chunks of which lie a multiple of 4 KB apart: the chunks are
    one word longer (the first) or 61 words (the second)."""
    torch = torch_cuda()
    import paper_2009_03254_amd as bc
    f = _field("plane", dims, 0)
    iso = np.float32(100.0)
    say(f"[dense chunks] {dims}")
    dm = bc.DenseMC(dims)
    v, vb = orc.mc_extract_dense(f, iso)
    out = torch.full((len(vb) + 8, 4), -7, dtype=torch.int32, device="cuda")
    rc, T = dm.extract_into(to_cuda(f), float(iso), out)
    assert rc == 0 and 3 * T == len(vb)
    got = out.cpu().numpy()
    assert np.array_equal(got[: 3 * T, :3].view(np.uint32), v.view(np.uint32))
    assert np.array_equal(got[: 3 * T, 3].view(np.uint32), vb)
    assert (got[3 * T:] == -7).all()
    dm.close()
