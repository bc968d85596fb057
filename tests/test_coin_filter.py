"""The binary32 coin filter of the simulation kernel: a coin whose sign lies
outside the filter's margin must equal the binary64 threshold's, over the
parameter and covariate ranges the filter takes (CPU), and whole simulations
with per-trial thresholds must equal the oracle's where the filter has to
leave every coin to the threshold or sits at its limits (GPU)."""
import numpy as np
import pytest

import oracle
from gpu_util import SEED, compare_with_oracle, say
from paper_1701_03549_amd import synth

LOG2E = 1.4426950408889634074
F = np.float32


def _fma(a, b, c):
    # the product of two binary32 values is exact in binary64; one more
    # rounding than a fused step, so no smaller an error
    return (a.astype(np.float64) * b + c).astype(F)


def _filter(beta, forest, psi, wind_deg, slope, up, d, r, ulp):
    """coin_margin and filter_beta in numpy: (s, margin); ulp scales 2^x by
    1 + ulp * 2^-23 (the instruction's last place)."""
    b = [(-LOG2E * beta[:, i]).astype(F) for i in range(5)]
    b3r = (-LOG2E * np.sqrt(0.5) * beta[:, 3]).astype(F)
    b4 = (-LOG2E / 8388608.0 * beta[:, 4]).astype(F)
    rad = np.deg2rad(wind_deg.astype(np.float64))
    cw, sw = np.cos(rad).astype(F), np.sin(rad).astype(F)
    s4 = np.where(d < 4, F(1), F(-1))
    wind = np.select([d % 4 == 0, d % 4 == 1, d % 4 == 2], [s4 * b[3] * cw, s4 * b3r * (cw + sw), s4 * b[3] * sw],
                     s4 * b3r * (sw - cw)).astype(F)
    x = b[0] + np.where(forest, b[1], F(0))
    x = _fma(b[2], psi.astype(F), x) + wind
    x = _fma(b4, np.where(up, np.rint(slope * 8388608.0), 0.0).astype(F), x)
    u = _fma(r.astype(F), F(2.0 ** -32), F(2.0 ** -33))
    with np.errstate(over="ignore", under="ignore"):
        e = (np.exp2(x.astype(np.float64)) * (1.0 + ulp * 2.0 ** -23)).astype(F)
        s = _fma(u, e, u) - F(1)
    total = np.abs(beta).sum(axis=1)
    return s, np.where(total < 1e4, (total + 1.0) / 524288.0, np.inf)


@pytest.mark.parametrize("scale", [0.01, 1.0, 5.0, 30.0, 1000.0])
@pytest.mark.parametrize("near", [True, False])
def test_filter_agrees_with_the_threshold(scale, near):
    rng = np.random.default_rng(int(scale * 100) + near)
    n = 400_000
    beta = rng.normal(0.0, scale, size=(n, 5))
    forest, up = rng.random(n) < 0.4, rng.random(n) < 0.5
    psi = np.where(rng.random(n) < 0.3, 0.0, rng.uniform(-1, 1, n))
    wind = rng.uniform(-400, 400, n).astype(F)
    slope = (rng.uniform(0, 89.9, n).astype(F)).astype(np.float64) / 100.0
    d = rng.integers(0, 8, n)
    omega = np.cos((wind.astype(np.float64) - 45.0 * d) * np.pi / 180.0)
    x = beta[:, 0] + beta[:, 1] * forest + beta[:, 2] * psi + beta[:, 3] * omega + beta[:, 4] * np.where(up, slope, 0)
    with np.errstate(over="ignore"):
        t = np.rint(1.0 / (1.0 + np.exp(-np.clip(x, -40, 40))) * 2.0 ** 32)
    r = rng.integers(0, 2 ** 32, n).astype(np.float64)
    if near:  # coins at and around the threshold, to relative distances of 2^-30 .. 2^-8
        r = np.clip(np.rint(t * (1.0 + rng.choice([-1, 1], n) * 2.0 ** -rng.uniform(8, 30, n))), 0, 2 ** 32 - 1)
        r[: n // 8] = np.clip(t[: n // 8] + rng.integers(-1, 2, n // 8), 0, 2 ** 32 - 1)
    hit = (t >= 2.0 ** 32 - 1) | (r < t)
    for ulp in (-2, 2):
        s, margin = _filter(beta, forest, psi, wind, slope, up, d, r, ulp)
        sure = np.abs(s) > margin
        assert np.array_equal(hit[sure], (s < 0)[sure])
        if not near:  # the filter decides almost every coin
            assert np.mean(~sure) < 4e-6 * (1.0 + 5.0 * scale)


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["steep", "windy", "huge", "zero", "saturated"])
def test_per_trial_coins_at_the_filters_limits(case):
    """Slopes outside [0, 100) and wind angles beyond exact reduction (cells
    the filter marks), parameters beyond its range, all-zero parameters and
    saturated thresholds: per-trial runs equal the oracle's."""
    from paper_1701_03549_amd import fire
    say(f"coin filter {case}")
    W, H, n = 75, 50, 6
    ls = synth.random_small_landscape(W, H, 31)
    beta = (-1.0, 0.5, 0.4, 0.8, 0.3)
    if case == "steep":
        ls["slope_deg"][::3] = 180.0
        ls["slope_deg"][1::5, ::2] = -40.0
    elif case == "windy":
        ls["wind_to_deg"][::2] = 3.0e9
        ls["wind_to_deg"][1::4] = -1234.5
    elif case == "huge":
        beta = (1e39, -1e39, 3e38, 2.0, -7e5)
    elif case == "zero":
        beta = (0.0,) * 5
    else:
        beta = (25.0, -60.0, 1.0, 1.0, 1.0)
    T = oracle.thresholds(ls, beta)
    ign = synth.nearest_burnable(ls["veg"], W // 2, H // 2)
    g = fire.FireGPU(0)
    try:
        lid = g.load_landscape(ls)
        # the covariates' cosines differ by an ulp between libraries: the library's own table
        Tg = g.thresholds(lid, beta).cpu().numpy().view(np.uint32)
        assert np.abs(Tg.astype(np.int64) - T.astype(np.int64)).max() <= 1 or case == "windy"
        sims = fire.make_sims(n, lid, -1, ign)
        for threads in (64, 256):
            g.set_schedule(threads=threads, queue_cap=128, table_mode=0, wg_per_cu=2)
            res, maps = g.run([beta], sims, SEED, want_maps=True)
            g.sync()
            compare_with_oracle(ls, [Tg], fire.results_to_numpy(res), maps.cpu().numpy().view(np.uint32), sims, SEED)
    finally:
        g.close()
