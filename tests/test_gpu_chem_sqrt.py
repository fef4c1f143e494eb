"""The square root of T in the cooling, rounded as IEEE rounds it. In fully ionised hydrogen at
1e13 to 1e15 K only bremsstrahlung is left of the cooling and its Gaunt factor is 1.1, so one
sub-step that takes all but a thousandth of the energy away turns the last bit of the root into
6e-5 of the final temperature, against 2^-22 allowed (the FP32 rounding of that temperature, and
the recombination of 3e-8 of the gas)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

K_B = 1.380649e-16


def test_bremsstrahlung_takes_the_rounded_root(arc):
    import torch

    f = np.float32
    shape, left = (64, 64, 64), 1e-3
    rng = np.random.default_rng(3)
    T = (10.0 ** rng.uniform(13, 15, shape)).astype(f)
    n_h = (1e-3 * np.sqrt(T.astype(np.float64) / 1e14)).astype(f)  # the same cooling time everywhere
    rate = (f(1.42e-27) * f(1.1)) * np.sqrt(T)  # FP32 operations
    assert rate.dtype == f
    nh, temp = n_h.astype(np.float64), T.astype(np.float64)
    energy = 3.0 * K_B * temp * nh
    dt = (1.0 - left) * np.median(energy / (rate * nh * nh))
    expect = temp * (1.0 - rate * nh * nh * dt / energy)
    near = np.abs(expect / temp / left - 1.0) < 0.5
    assert near.mean() > 0.9
    zero = torch.zeros(shape, device="cuda")
    g = {"n_h": torch.from_numpy(n_h).cuda(), "x_hi": zero.clone(), "x_hei": zero.clone(), "x_heii": zero.clone(),
         "temp": torch.from_numpy(T).cuda(), "cell_cm": 1e21, "y_he": 0.0}
    rates = torch.zeros((3,) + shape, device="cuda")
    ctx = arc.Context(0)
    try:
        st = ctx.chem_step(g, rates, rates.clone(), dt, eps=1e30, max_sub=4)
    finally:
        ctx.close()
    assert st["sub_total"] == T.size
    err = np.abs(g["temp"].cpu().numpy()[near] / expect[near] - 1.0)
    print(f"[sqrt] largest {err.max():.2e}, share above 2^-22 {np.mean(err > 2.0 ** -22):.4f}")
    assert err.max() <= 2.0 ** -22
