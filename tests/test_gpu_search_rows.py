"""Row reads and maximum search at the edges of their ranges (needs an MI355X).

Integer-valued cubes searched as they are: every sum is exact in any order, and
small values make many windows tie, so S/N is the oracle's up to the rounding
of the normaliser and of the quotient (2^-22 relative) and every TOA is the
first window that reaches the maximum.
"""
import numpy as np
import pytest

from oracle import search as osr
from paper_2510_18136_amd import nsfrb
from tests._lib import ensure_built

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"


def check(nt, ns, store, widths, dms, nx=3, ny=2):
    rng = np.random.default_rng(nt * 100 + ns)
    cube = rng.integers(-3, 4, (nt, ns, nx * ny)).astype(np.float32)
    cube[:, :, 1] = 1.0                                   # every window of a width ties
    cfg = nsfrb.SearchConfig(nx, ny, nt, np.linspace(1.311, 1.499, ns), dms, widths, in_dtype=store,
                             store_dtype=store, norm="none", snr_threshold=1e9, max_candidates=4)
    x = torch.from_numpy(cube).to(TORCH[store]).cuda()
    with nsfrb.Search(cfg) as s:
        info = s.plan_info()
        print(f"[gpu] rows nt={nt} ns={ns} store={store} plan={info}", flush=True)
        s.run(x.data_ptr(), torch.cuda.current_stream().cuda_stream)
        s.candidates()
        snr, toa = s.maps()
        delays = s.delay_table()
    want, want_toa = osr.snr_toa_maps(cube.astype(np.float64), delays, list(widths))
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(snr), fin)
    assert (np.abs(snr[fin] - want[fin]) <= 2.0 ** -22 * np.abs(want[fin])).all()
    np.testing.assert_array_equal(toa, want_toa)
    return (info["row_len"] - 1 - delays.max()) // 64      # samples per lane


# around every change of samples per lane: one, the first grouped maximum search
# (17), rows read in halves (20 and more), odd and paired rows
@pytest.mark.parametrize("store", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("nt", [63, 64, 127, 700, 1000, 1087, 1088, 1215, 1279, 1500, 2047, 2048])
def test_row_lengths(nt, store):
    widths = [w for w in (1, 2, 4, 8, 16, 23, 64, 300, 1024) if w <= nt]
    check(nt, 5, store, widths, np.linspace(0.0, 4000.0, 9))


@pytest.mark.parametrize("store,ns,c", [("f32", 18, 34), ("f32", 19, 33), ("bf16", 37, 34), ("bf16", 38, 33)])
def test_paired_rows_only_where_they_fit(store, ns, c):
    assert check(2048, ns, store, [1, 2, 4, 8], np.linspace(0.0, 500.0, 3), nx=2, ny=1) == c


def test_lean_plan():
    """A long series with many widths: the plan that spends the fewest registers."""
    check(2400, 4, "f32", list(range(1, 18)), np.linspace(0.0, 1000.0, 4), nx=2, ny=1)


@pytest.mark.parametrize("store,nt,c", [("f32", 2048, 34), ("f32", 2176, 35), ("f16", 2048, 34), ("bf16", 2048, 34),
                                        ("bf16", 700, 11), ("f32", 333, 6)])
def test_plan_info_names_the_samples_per_lane_that_run(store, nt, c):
    cfg = nsfrb.SearchConfig(3, 2, nt, np.linspace(1.311, 1.499, 5), np.linspace(0.0, 500.0, 3), [1, 2, 4], store_dtype=store)
    with nsfrb.Search(cfg) as s:
        info, dmax = s.plan_info(), int(s.delay_table().max())
    assert info["samples_per_lane"] == (info["row_len"] - 1 - dmax) // 64 == c
