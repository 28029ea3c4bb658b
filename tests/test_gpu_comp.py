"""GPU parity for the compensation of the diagonal noise model (Section
3.2): the per-(frequency, time) factor and the rounding that uses it equal
the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1503_00638_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = synth.N_SAMPLES_DEFAULT


@pytest.fixture(scope="module")
def bsg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_00638_amd as m
    m.load()
    return m


def dev(a):
    return torch.from_numpy(np.array(a, copy=True, order="C")).to("cuda:0")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# Up to 6 inputs a thread takes a sample, above that a workgroup takes one
# frequency's products (T = 2 with 40 inputs: many rows of products per step).
CASES = [(4, 8, 64, 0, 0.4), (3, 5, 7, 1, 0.0), (2, 16, 130, 2, 2.0), (1, 1, 5, 3, 0.4),
         (2, 2, 65, 4, 1.0), (5, 3, 1, 5, 0.4), (16, 8, 64, 6, 0.1), (2, 40, 2, 7, 0.4),
         (1, 4, 1024, 8, 0.4), (3, 13, 32, 9, 0.0)]


@pytest.mark.parametrize("F,I,T,seed,source", CASES)
def test_compensation_factor_parity(bsg, F, I, T, seed, source):
    vis, autos = synth.gen_vis_point_source(F, I, T, seed, source)
    ref = oracle.noise_compensation(vis, autos)
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


@pytest.mark.parametrize("F,I,T,seed,source", CASES)
def test_compensated_rounding_parity(bsg, F, I, T, seed, source):
    vis, autos = synth.gen_vis_point_source(F, I, T, seed, source)
    m = oracle.noise_compensation(vis, autos)
    for f in (0.01, 1e-3):
        ref = oracle.round_to_noise_scaled(vis, autos, N, f, m)
        got = host(bsg.round_to_noise_scaled(dev(vis), dev(autos), N, f, dev(m)))
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), f
    # the device factor feeds the device rounding directly
    dv, da = dev(vis), dev(autos)
    got = host(bsg.round_to_noise_scaled(dv, da, N, 0.01, bsg.noise_compensation(dv, da)))
    assert np.array_equal(got.view(np.uint32), oracle.round_to_noise_scaled(vis, autos, N, 0.01, m).view(np.uint32))


@pytest.mark.parametrize("T", [40, 32])
def test_compensation_degenerate_inputs(bsg, T):
    vis, autos = synth.gen_vis_point_source(3, 6, T, 9, 0.4)
    autos[0, 1, :5] = [0.0, -3.0, np.nan, np.inf, 1e-40]
    autos[1, :, 7] = 0.0
    vis.view(np.float32).reshape(-1)[::17] = np.nan
    ref = oracle.noise_compensation(vis, autos)
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
    ref_r = oracle.round_to_noise_scaled(vis, autos, N, 0.01, ref)
    got_r = host(bsg.round_to_noise_scaled(dev(vis), dev(autos), N, 0.01, dev(ref)))
    assert np.array_equal(got_r.view(np.uint32), ref_r.view(np.uint32))


@pytest.mark.parametrize("F,I,T", [(1, 128, 32), (2, 40, 1), (3, 12, 513), (1, 9, 1100), (2, 61, 50),
                                   (1, 200, 7), (600, 3, 5), (1, 512, 32)])
def test_compensation_shapes_and_scales(bsg, F, I, T):
    """Products over several workgroups, times of every kind, and a float32
    screening that has to let every product through that matters: autos and
    visibilities over 60 decades (products that overflow or underflow in
    float32), correlations of nearly 1, repeated minima, zero, negative,
    infinite and NaN values."""
    rng = np.random.default_rng(F * 1000 + I + T)
    vis, autos = synth.gen_vis_point_source(F, I, T, 5, 0.4)
    g = (10.0 ** rng.uniform(-15, 15, (F, I, T))).astype(np.float32)
    pairs = synth.product_pairs(I)
    with np.errstate(over="ignore", under="ignore", invalid="ignore"):
        vis = (vis * np.sqrt(g[:, pairs[:, 0]]) * np.sqrt(g[:, pairs[:, 1]])).astype(np.complex64)
        autos = (autos * g).astype(np.float32)
    flat = autos.reshape(-1)
    for v in (0.0, -1.0, np.inf, np.nan, 1e38, 1e-40):
        flat[rng.integers(0, flat.size, max(1, flat.size // 97))] = v
    vflat = vis.view(np.float32).reshape(-1)
    for v in (0.0, np.inf, np.nan, 1e38, 1e-40):
        vflat[rng.integers(0, vflat.size, max(1, vflat.size // 199))] = v
    ref = oracle.noise_compensation(vis, autos)
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


def test_unit_scale_is_plain_rounding(bsg):
    vis, autos = synth.gen_vis(4, 8, 64, 0)
    ones = torch.ones((4, 64), dtype=torch.float64, device="cuda:0")
    a = host(bsg.round_to_noise_scaled(dev(vis), dev(autos), N, 0.01, ones))
    b = host(bsg.round_to_noise(dev(vis), dev(autos), N, 0.01))
    assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_compensation_prod_map(bsg):
    vis, autos = synth.gen_vis_point_source(2, 5, 16, 10, 0.4)
    P = vis.shape[1]
    pm = np.ascontiguousarray(synth.product_pairs(5)[np.random.default_rng(2).permutation(P)])
    ref = oracle.noise_compensation(vis, autos, prod_map=pm)
    got = host(bsg.noise_compensation(dev(vis), dev(autos), prod_map=dev(pm)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


@pytest.mark.parametrize("I,T", [(64, 32), (128, 7), (256, 32)])
@pytest.mark.parametrize("ab,ratio", [(1e-45, 1e15), (3e-42, 1e12), (1e-39, 1e9), (1e-38, 1e9)])
def test_compensation_subnormal_auto_products(bsg, I, T, ab, ratio):
    """V_ii V_jj below the normal float32 range under cross products far above
    it: the float32 product is off by up to a half there, so it must not decide
    which terms can be the minimum.  Every time has its first products near the
    lowest term and hundreds of later ones just above and below it."""
    rng = np.random.default_rng(I + T)
    P = I * (I + 1) // 2
    autos = (np.sqrt(ab) * 10.0 ** rng.uniform(-0.5, 0.5, (2, I, T))).astype(np.float32)
    pairs = synth.product_pairs(I)
    prod = autos[:, pairs[:, 0]].astype(np.float64) * autos[:, pairs[:, 1]].astype(np.float64)
    r = ratio * rng.uniform(1.0, 1.3, (2, P, T))
    vis = np.sqrt(r * prod).astype(np.complex64)
    ref = oracle.noise_compensation(vis, autos)
    assert (ref < -0.9 * ratio).all()
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


@pytest.mark.parametrize("lo,hi", [(-45, 38), (-24, -18), (-20, 19)])
def test_compensation_over_the_float32_range(bsg, lo, hi):
    """Autos and visibilities each anywhere in the float32 range (subnormal
    ones too), independent of each other."""
    rng = np.random.default_rng(hi - lo)
    F, I, T = 3, 96, 32
    P = I * (I + 1) // 2
    with np.errstate(over="ignore", under="ignore"):
        autos = (10.0 ** rng.uniform(lo, hi, (F, I, T))).astype(np.float32)
        vis = (10.0 ** rng.uniform(lo, hi, (F, P, T, 2))).astype(np.float32)
    vis = vis.view(np.complex64)[..., 0]
    ref = oracle.noise_compensation(vis, autos)
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


@pytest.mark.parametrize("F,I,T,seed", [(30000, 2, 7, 1), (40000, 6, 1, 2), (5000, 6, 64, 3), (1, 7, 3, 4),
                                        (18725, 7, 7, 5), (18724, 7, 7, 6), (1033, 9, 127, 7), (1008, 9, 130, 8),
                                        (300, 10, 129, 9), (2, 24, 64, 10), (256, 12, 128, 11),
                                        (257, 12, 128, 12), (200000, 1, 3, 13), (4400000, 2, 1, 14)])
def test_compensation_small_arrays(bsg, F, I, T, seed):
    """Few products over many samples, on both sides of each rule that picks
    the kernel, its threads and its times."""
    rng = np.random.default_rng(seed)
    P = I * (I + 1) // 2
    autos = rng.uniform(0.5, 2.0, (F, I, T)).astype(np.float32)
    vis = rng.uniform(-0.4, 0.4, (F, P, T, 2)).astype(np.float32).view(np.complex64)[..., 0]
    for v in (0.0, -1.0, np.inf, np.nan, 1e-40):
        autos.reshape(-1)[rng.integers(0, autos.size, max(1, autos.size // 501))] = v
    pm = np.ascontiguousarray(synth.product_pairs(I)[rng.permutation(P)])
    ref = oracle.noise_compensation(vis, autos)
    got = host(bsg.noise_compensation(dev(vis), dev(autos)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
    ref = oracle.noise_compensation(vis, autos, prod_map=pm)
    got = host(bsg.noise_compensation(dev(vis), dev(autos), prod_map=dev(pm)))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


@pytest.mark.parametrize("I", [16384, 16385])
def test_compensation_largest_arrays(bsg, I):
    """The most inputs whose autos have a place in LDS, and one more."""
    P = I * (I + 1) // 2
    g = torch.Generator(device="cuda:0").manual_seed(I)
    v = torch.rand((1, P, 1, 2), generator=g, device="cuda:0") * 0.6 - 0.3
    a = torch.rand((1, I, 1), generator=g, device="cuda:0") + 0.5
    vis = torch.view_as_complex(v)
    ref = oracle.noise_compensation(host(vis), host(a))
    got = host(bsg.noise_compensation(vis, a))
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
