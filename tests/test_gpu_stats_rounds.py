"""Noise statistics at the edges of the selection and of its tiles (needs an MI355X).

Median, sigma and normalised cube are compared bit for bit: the two middle
samples and distances are selected, never summed, and sigma, the quotient and
its rounding are single correctly rounded FP64 operations on both sides.
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


def check(cube, nx, ny, raw="f32", store="f32"):
    x = torch.from_numpy(np.ascontiguousarray(cube, dtype=np.float32)).to(TORCH[raw])
    nt, ns = cube.shape[:2]
    cfg = nsfrb.SearchConfig(nx, ny, nt, np.linspace(1.311, 1.499, ns), [0.0], [1], in_dtype=raw, store_dtype=store,
                             snr_threshold=1e9, max_candidates=4)
    print(f"[gpu] stats nt={nt} ns={ns} pixels={nx * ny} raw={raw} store={store}", flush=True)
    d = x.cuda()
    with nsfrb.Search(cfg) as s:
        s.run(d.data_ptr(), torch.cuda.current_stream().cuda_stream)
        s.candidates()
        med, sig = s.noise_stats()
        z, flags = s.zcube()[0], s.flag_count()
    want_z, want_med, want_sig, want_flags = osr.normalize(x.float().numpy(), store=store)
    np.testing.assert_array_equal(med.reshape(nx * ny, ns), want_med)
    np.testing.assert_array_equal(sig.reshape(nx * ny, ns), want_sig)
    np.testing.assert_array_equal(np.asarray(z, np.float64).reshape(nx * ny, ns, nt), want_z.transpose(2, 1, 0))
    assert flags == want_flags


# every register class and the remainders of its four-sample groups; 21 pixels:
# the last tile is moved back over the one before it
@pytest.mark.parametrize("raw,store", [("f32", "f32"), ("f16", "bf16"), ("bf16", "f16")])
@pytest.mark.parametrize("nt", [1, 2, 3, 64, 65, 127, 128, 129, 255, 256, 257, 509, 512, 513, 1023, 1025, 1530, 2046,
                                2048, 2049, 4093, 4096])
def test_lengths(nt, raw, store):
    rng = np.random.default_rng(nt)
    check(rng.standard_normal((nt, 2, 21)) * 1.7 + 0.3, 7, 3, raw, store)


@pytest.mark.parametrize("raw", ["f32", "f16"])
@pytest.mark.parametrize("n_pix", [1, 5, 15, 16, 17, 31, 33])
def test_planes_around_a_tile(n_pix, raw):
    rng = np.random.default_rng(n_pix)
    check(rng.standard_normal((300, 3, n_pix)), n_pix, 1, raw)


def values(kind, nt, shape, rng):
    g = rng.standard_normal(shape)
    if kind == "outliers":                    # a crowded bin: binned again
        g[rng.integers(0, nt, 3)] += 5000.0
    elif kind == "nested":                    # several rounds
        g[: nt // 8] *= 1e6
        g[nt // 8: nt // 4] *= 1e3
    elif kind == "offset":                    # the median is no FP32 value: distances need the check
        g += 4096.0
    elif kind == "levels":                    # a few values shared by many samples
        g = np.round(g) + 1000.0
    elif kind == "two":                       # MAD of half the gap
        g = np.where(np.arange(nt)[:, None, None] % 2 == 0, 1.25, 2.0) + 0.0 * g
    elif kind == "flat":                      # MAD 0: unusable
        g = np.where(g > 1.5, g, 0.5)
    elif kind == "one_lane":                  # the middle values all fall to one lane
        t = np.arange(nt)
        mid = (t % 256) // 4 == 5
        g = np.where(mid[:, None, None], 1e-3 * g, 10.0 * np.sign(g) + g)
    elif kind == "huge":                      # the range overflows FP32
        g *= 3e37
        g[0], g[1] = 3e38, -3e38
    elif kind == "ramp":
        g = np.arange(nt, dtype=np.float64)[:, None, None] * 0.01 + 0.0 * g
    return g


@pytest.mark.parametrize("nt", [200, 333, 1000, 2047, 2048])
@pytest.mark.parametrize("kind", ["outliers", "nested", "offset", "levels", "two", "flat", "one_lane", "huge", "ramp"])
def test_value_distributions(kind, nt):
    rng = np.random.default_rng(nt)
    check(values(kind, nt, (nt, 2, 48), rng), 8, 6)


def edge_series(n, edge):
    """64 series [64][n] whose MAD rank lies at the edge of a crowded bin of distances.

    The median is 1 + 2^-24, halfway between two FP32 values, and distances are taken from the FP32 value 1: a
    sample below has an FP64 distance 2^-24 more than its key, one above 2^-24 less. Around the edge lie a key 2^-24
    short of 0.3 from below the median and the key 0.3 from above it, whose order the FP64 distances reverse. The
    outlier, which sets the bins, sweeps 64 consecutive FP32 values, so that a bin's edge falls between the two keys
    for some of them.
    """
    u, half, rng = 2.0 ** -24, n // 2, np.random.default_rng(n)
    key = round(0.3 / (2 * u)) * 2 * u

    def below(m, lo, hi):
        return 1.0 - np.round(rng.uniform(lo, hi, m) / u) * u

    def above(m, lo, hi):
        return 1.0 + np.round(rng.uniform(lo, hi, m) / (2 * u)) * 2 * u

    if edge == "lower":                       # the first key of bin 1
        q, far = half - n // 8, np.float32(key * 1020 / 3.5)
        x = [[1.0, 1.0 - (key - u)], below(q - 2, 0.01, 0.25), below(n // 8, key + 0.01, key + 0.2),
             [1.0 + 2 * u], above(n // 8 - 2, 0.01, 0.25), [1.0 + key], above(half - n // 8 - 1, key + 0.01, key + 0.2)]
    else:                                     # the last key of bin 1
        q, far = n // 16 + n // 4, np.float32(key * 1020 / 7.5)
        x = [[1.0], below(n // 16 - 1, 0.01, 0.12), below(n // 4 - 1, 0.16, 0.28), [1.0 - (key - u)],
             below(half - q, 0.31, 0.5), [1.0 + 2 * u], above(half - q, 0.16, 0.28), [1.0 + key],
             above(q - 3, 0.31, 0.5)]
    outlier = 1.0 + (np.float64(far) + (np.arange(64) - 32) * np.float64(np.spacing(far)))
    return np.concatenate([np.repeat(np.concatenate(x)[None], 64, 0), outlier[:, None]], axis=1)


@pytest.mark.parametrize("nt", [256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("edge", ["lower", "upper"])
def test_rank_at_the_edge_of_a_crowded_bin(nt, edge):
    x = edge_series(nt, edge)
    assert x.shape == (64, nt) and (x == x.astype(np.float32)).all()
    assert (np.median(x, axis=1) == 1.0 + 2.0 ** -24).all()
    check(x.T[:, None], 8, 8)


@pytest.mark.parametrize("nt", [1, 64, 500, 700, 1024, 2047, 2048, 4096])
def test_equal_samples(nt):
    """Selection takes no histogram round for them: nothing of one may be used after it. Beside them, ordinary series."""
    rng = np.random.default_rng(nt)
    x = rng.standard_normal((nt, 2, 32))
    x[:, :, ::2] = rng.choice([0.0, -0.0, 1.0, -3.7e30, 1e-42, 4096.5], (1, 2, 16))
    check(x, 8, 4)
