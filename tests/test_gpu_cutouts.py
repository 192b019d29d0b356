"""Cutout extraction at the edges of its tiles (needs an MI355X): exact values."""
import numpy as np
import pytest

from oracle import cnn
from paper_2510_18136_amd import nsfrb
from tests._lib import ensure_built

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"


# windows below, at and above the 64 times of a tile; images and series smaller
# than a cutout and larger; candidates outside on every side
@pytest.mark.parametrize("store", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny,nt,ct", [(40, 37, 150, 1), (9, 5, 33, 63), (33, 50, 64, 64), (40, 40, 200, 65),
                                         (1, 1, 1, 130)])
def test_cutouts_exact(nx, ny, nt, ct, store):
    rng = np.random.default_rng(nt + ct)
    ns = 16
    z = [torch.from_numpy(rng.standard_normal((nx * ny, ns, nt)).astype(np.float32)).to(TORCH[store]) for _ in range(2)]
    delays = rng.integers(0, nt, (3, ns)).astype(np.int32)
    descs = [(0, nx // 2, ny // 2, 1, nt // 2), (1, 0, ny - 1, 2, 0), (1, nx - 1, 0, 0, nt - 1), (0, -40, 3, 1, 5),
             (1, 0, 0, 2, -2 * nt - ct), (0, nx + 15, ny + 15, 0, 3 * nt)]
    zd = [v.cuda() for v in z]
    n = len(descs)
    # at an odd sample of the buffer, with guards on both sides
    buf = torch.full((1 + n * ct * 32 * 32 * ns + 1,), 0x7abc, dtype=torch.int16, device="cuda")
    print(f"[gpu] cutouts nx={nx} ny={ny} nt={nt} ct={ct} store={store}", flush=True)
    with nsfrb.Classifier(max_batch=n, n_time=ct, ny=32) as c:
        c.cutouts([v.data_ptr() for v in zd], store, nx, ny, ns, nt, delays, descs, buf.data_ptr() + 2,
                  stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    raw = buf.cpu().numpy()
    assert raw[0] == 0x7abc and raw[-1] == 0x7abc
    got = (raw[1:-1].view(np.uint16).astype(np.uint32) << 16).view(np.float32).reshape(n, ct, 32, 32, ns)
    for k, (cube, px, py, d, toa) in enumerate(descs):
        xi, yi = px + np.arange(32) - 16, py + np.arange(32) - 16
        t = toa - ct // 2 + np.arange(ct)[:, None] + delays[d][None, :]
        ok = (((yi >= 0) & (yi < ny))[None, :, None, None] & ((xi >= 0) & (xi < nx))[None, None, :, None]
              & ((t >= 0) & (t < nt))[:, None, None, :])
        pix = np.clip(yi, 0, ny - 1)[:, None] * nx + np.clip(xi, 0, nx - 1)[None, :]
        v = z[cube].float().numpy()[pix[None, :, :, None], np.arange(ns), np.clip(t, 0, nt - 1)[:, None, None, :]]
        np.testing.assert_array_equal(got[k], np.where(ok, cnn.bf16(v).astype(np.float32), np.float32(0)))
