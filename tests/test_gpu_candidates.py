"""Candidate lists at the edges of their kernels (needs an MI355X).

One sample, one sub-band, one DM and width 1: a pixel's best S/N is its own
sample, so every list is known exactly. Sizes lie at one pixel per thread
block, at the changes of pixels per thread and at the longest list that is
merged; values are distinct, tied at the K-th place, all equal, or all below
the threshold.
"""
import numpy as np
import pytest

from paper_2510_18136_amd import nsfrb
from tests._lib import ensure_built

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"


def config(nx, ny, k, theta):
    return nsfrb.SearchConfig(nx, ny, 1, [1.4], [0.0], [1], norm="none", snr_threshold=theta, max_candidates=k)


def values(kind, n, rng):
    if kind == "distinct":
        return rng.permutation(n).astype(np.float32) - n // 3          # both signs
    if kind == "ties":
        return rng.integers(0, 3, n).astype(np.float32)
    if kind == "equal":
        return np.full(n, 7.0, np.float32)
    return np.full(n, -1e6, np.float32)                                # below


def expected(v, theta, k, nx):
    hit = np.flatnonzero(v >= theta)
    order = hit[np.lexsort((hit, -v[hit]))][:k]
    return [(int(p) % nx, int(p) // nx, float(v[p])) for p in order], hit.size


def got(s):
    recs, total, _ = s.candidates()
    assert all(r["dm_index"] == 0 and r["width_index"] == 0 and r["toa"] == 0 for r in recs)
    return [(r["x"], r["y"], r["snr"]) for r in recs], total


@pytest.mark.parametrize("nx,ny,k", [(1, 1, 1), (255, 1, 10), (16, 16, 10), (1025, 1, 10), (64, 64, 16),
                                     (201, 150, 100), (256, 256, 256), (256, 256, 257), (700, 600, 10),
                                     (128, 128, 4096)])
@pytest.mark.parametrize("kind", ["distinct", "ties", "equal", "below"])
def test_lists(nx, ny, k, kind):
    v = values(kind, nx * ny, np.random.default_rng(nx + k))
    theta = -50.0 if kind == "distinct" else 1.0
    x = torch.from_numpy(v).cuda()
    with nsfrb.Search(config(nx, ny, k, theta)) as s:
        print(f"[gpu] candidates {nx}x{ny} K={k} {kind}", flush=True)
        for _ in range(2):                             # the counters are left ready for the next run
            s.run(x.data_ptr())
            assert got(s) == expected(v, theta, k, nx)


def test_flag_count_of_each_run():
    v = np.zeros(4096, np.float32)
    bad = v.copy()
    bad[[3, 77, 4095]] = np.nan
    with nsfrb.Search(config(64, 64, 10, 1.0)) as s:
        for cube, n in ((bad, 3), (v, 0), (bad, 3), (bad, 3)):
            x = torch.from_numpy(cube).cuda()
            s.run(x.data_ptr())
            assert s.flag_count() == n


def test_batch_lists():
    """Cubes of every size in one launch, graph replays with other values in between."""
    rng = np.random.default_rng(9)
    shapes = [(1, 1), (33, 31), (64, 64), (200, 150), (300, 300)]
    cfgs = [config(nx, ny, 12, 1.0) for nx, ny in shapes]
    xs = [torch.zeros(nx * ny, device="cuda") for nx, ny in shapes]
    with nsfrb.Batch(cfgs) as b:
        for kind in ("ties", "below", "equal", "ties"):
            vs = [values(kind, nx * ny, rng) for nx, ny in shapes]
            for x, v in zip(xs, vs):
                x.copy_(torch.from_numpy(v))
            torch.cuda.synchronize()
            b.run([x.data_ptr() for x in xs])
            for i, (nx, ny) in enumerate(shapes):
                recs, total = b.candidates(i)
                assert ([(r["x"], r["y"], r["snr"]) for r in recs], total) == expected(vs[i], 1.0, 12, nx)


def test_runs_after_overlapping_ones():
    """Runs that overlap on two streams spoil each other only: the counters of the next run start at zero."""
    v = values("distinct", 256 * 256, np.random.default_rng(2))
    flagged = np.array([5, 9000, 65535])
    want = v.copy()
    want[flagged] = 0.0                                    # a flagged sample is searched as 0
    v[flagged] = np.nan
    x = torch.from_numpy(v).cuda()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    with nsfrb.Search(config(256, 256, 16, -50.0)) as s:
        print("[gpu] candidates, overlapping runs", flush=True)
        for _ in range(3):
            for st in streams * 8:
                s.run(x.data_ptr(), st.cuda_stream)
            torch.cuda.synchronize()
            s.run(x.data_ptr(), streams[0].cuda_stream)
            assert got(s) == expected(want, -50.0, 16, 256)
            assert s.flag_count() == flagged.size


@pytest.mark.parametrize("pinned", [True, False])
def test_best_maps_through_shared_or_no_pinned_memory(monkeypatch, pinned):
    """Cubes of one batch share a pinned buffer; maps too large for it, or all where none can be pinned, are copied singly."""
    if not pinned:
        monkeypatch.setenv("NSFRB_FORCE_PIN_FAIL", "1")
    rng = np.random.default_rng(4)
    shapes = [(5, 3), (520, 510), (512, 512), (64, 64)]
    vs = [values("distinct", nx * ny, rng) for nx, ny in shapes]
    xs = [torch.from_numpy(v).cuda() for v in vs]
    with nsfrb.Batch([config(nx, ny, 4, 1e9) for nx, ny in shapes]) as b:
        b.run([x.data_ptr() for x in xs])
        for i in (3, 0, 2, 1):
            snr, d, w, t = b.best(i)
            np.testing.assert_array_equal(np.asarray(snr).ravel(), vs[i])
            assert not np.any(d) and not np.any(w) and not np.any(t)
    with nsfrb.Search(config(64, 64, 4, 1e9)) as s:
        s.run(xs[3].data_ptr())
        np.testing.assert_array_equal(np.asarray(s.best()[0]).ravel(), vs[3])
