"""The radiation-function tables as the FP64 steps read them: each kernel with
FP64 steps holds a window of a table in LDS and reads the cells outside it from
memory; qs_radiation_eval evaluates the forward table in memory."""
import math

import numpy as np
import pytest

from paper_2308_09348_amd import workloads

pytestmark = pytest.mark.gpu

ALPHA, LAMBDA_BAR_C, C = 7.2973525693e-3, 3.8615926796e-7, 0.299792458  # um, um/fs


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09348_amd as qs
    ctx = qs.Context(0)
    yield ctx
    ctx.close()


def _eval(gpu, chi):
    import torch
    return gpu.radiation_eval(torch.tensor(chi, device="cuda"), "fp64").cpu().numpy().T


def _integrate(gpu, p, g0):
    """The moment system of a plane-wave shot by RK4 on the host, with the
    radiation functions of qs_radiation_eval; also the chi values reached."""
    omega = 2.0 * np.pi * C / p["lambda_um"]
    aS = p["lambda_um"] / (2.0 * np.pi * LAMBDA_BAR_C)
    K, CD = 4.0 * ALPHA / (3.0 * aS), 55.0 / (6.0 * np.sqrt(3.0)) * ALPHA / aS ** 2
    wt = omega * p["tau_fs"]
    psi_max = p["window_fwhm"] * wt
    h = 2.0 * psi_max / p["n_steps"]
    reached = []

    def rhs(mu, s2, psi):
        a = abs(p["a0"] * np.exp(-2.0 * np.log(2.0) * (psi / wt) ** 2) * np.cos(psi))
        chi = 2.0 / aS * mu * a
        reached.append(chi)
        g, g1, g2, hq = _eval(gpu, chi)
        u = K * a * a
        return (-u * mu * mu * g - 0.5 * u * (2.0 * g + 4.0 * g1 + g2) * s2,
                -2.0 * u * mu * (2.0 * g + g1) * s2 + CD * a ** 3 * mu ** 4 * hq)

    mu, s2 = g0.copy(), np.zeros_like(g0)
    for j in range(p["n_steps"]):
        psi = -psi_max + j * h
        a, b = rhs(mu, s2, psi), None
        b = rhs(mu + 0.5 * h * a[0], s2 + 0.5 * h * a[1], psi + 0.5 * h)
        c = rhs(mu + 0.5 * h * b[0], s2 + 0.5 * h * b[1], psi + 0.5 * h)
        d = rhs(mu + h * c[0], s2 + h * c[1], psi + h)
        mu = mu + h / 6.0 * (a[0] + 2.0 * (b[0] + c[0]) + d[0])
        s2 = s2 + h / 6.0 * (a[1] + 2.0 * (b[1] + c[1]) + d[1])
    return mu, s2, np.concatenate(reached)


@pytest.mark.parametrize("precision,chi64", [("fp64", 0.0), ("fp32", 1e-30)])
def test_steps_use_the_evaluated_table(gpu, precision, chi64):
    """FP64 steps of the forward, tape and photon passes (a threshold below every
    chi: all of a mixed pass's steps) over chi from below 2^-12 to above 200, on
    both sides of every kernel's window, give the states of an integration with
    the values of qs_radiation_eval.  The two differ by roundings: 256 additions
    and some ten operations a step, relative to a state that loses energy
    (2^-53 each, and 2^-48 once where a mixed pass returns its FP32 pair)."""
    p = dict(workloads.plane_wave_1d(), a0=5.0, gamma0=8.0e6, sigma_gamma=1.0e5, tau_fs=1.0, window_fwhm=4.0,
             n_samples=200, n_steps=256, rr_model="quantum", deposit="gauss", e_hi=1.2e7,
             precision=precision, chi_fp64=chi64, n_ph=64, ph_lo=0.0, ph_hi=9.6e6)
    n = p["n_samples"]
    tape = gpu.new_tape(n)
    rec = gpu.forward(p, sample_stride=1, n_sample_records=n)["samples"].cpu().numpy()
    gpu.forward(p, tape=tape)
    g0 = rec[:, 7]
    mu, s2, chi = _integrate(gpu, p, g0)
    assert 200.0 < chi.max() < 256.0 and np.mean(chi < 2.0 ** -12) > 0.01
    for got in (rec[:, :2].T, tape[:2].cpu().numpy()):
        assert np.abs(got[0] / mu - 1.0).max() <= 2e-13
        assert np.abs(got[1] / s2 - 1.0).max() <= 2e-12
    loss = gpu.photons(p)["energy"].cpu().numpy()[1]
    assert abs(loss / (g0 - mu).sum() - 1.0) <= 2e-12


def _small_chi(chi, terms=9):
    """The functions of the derivative table (g and h with their derivatives) by
    their expansions in chi: with s = 3 chi y / 2,
      g = (9 sqrt3 / 8 pi) Int y   (1+s)^-3 F dy,
      h = (81 / 55 pi)     Int y^2 (1+s)^-4 F dy,
      F = (1/(1+s) + 1 + s) K_2/3(y) - Int_y K_1/3,
    the binomials expanded in s and the integrals by
    Int y^m K_nu dy = 2^(m-1) Gamma((m+1+nu)/2) Gamma((m+1-nu)/2)."""
    def k_moment(m, nu):
        return 2.0 ** (m - 1) * math.gamma((m + 1 + nu) / 2) * math.gamma((m + 1 - nu) / 2)

    def binomial(a, n):
        return math.prod((a - i) / (i + 1) for i in range(n))

    def series(power, q):
        return np.array([1.5 ** n * ((binomial(-q - 1, n) + binomial(-q + 1, n))
                                     * k_moment(power + n, 2 / 3)
                                     - binomial(-q, n) * k_moment(power + n + 1, 1 / 3)
                                     / (power + n + 1)) for n in range(terms)])

    g = 9.0 * math.sqrt(3.0) / (8.0 * math.pi) * series(1, 3)
    h = 81.0 / (55.0 * math.pi) * series(2, 4)
    n = np.arange(terms)
    x = chi[:, None] ** n
    return np.stack([x @ g, x @ (n * g), x @ (n * (n - 1) * g), x @ h,
                     x @ (n * (n - 1) * (n - 2) * g), x @ (n * h)])


def test_tables_at_small_chi(gpu):
    """The FP64 tables below chi = 2^-11 (through the even cells below 2^-12 and
    on both sides of their ends) are at the rounding of their nodes: sums of 583
    terms that are sums of up to 600, sqrt(583 * 600) roundings of 2^-53, times the
    sum of the magnitudes combined (I_k = (k+1)! I_0 at small chi: 1, I_1 + 2 I_0 =
    4, 24, 192; J_1 + 3 J_0 = 6).  (One cubic over [0, 2^-12) is off by 1.5e-13,
    6.2e-13, 1.8e-12, 1.3e-12 of g, chi g', chi^2 g'', h and by 5.1e-12 of chi h'.)"""
    import torch
    edges = np.arange(1, 17) * 2.0 ** -16
    chi = np.concatenate([np.exp(np.linspace(math.log(1e-9), math.log(2.0 ** -11), 997)),
                          edges * (1 - 2.0 ** -50), edges, edges * (1 + 2.0 ** -50)])
    ref = _small_chi(chi)
    tol = math.sqrt(583 * 600) * 2.0 ** -53 * np.array([1.0, 4.0, 24.0, 1.0, 192.0, 6.0])
    err = np.abs(_eval(gpu, chi) - ref[:4]).max(axis=1)
    assert np.all(err <= tol[:4]), err
    d = gpu.radiation_derivs(torch.tensor(chi, device="cuda"), "fp64").cpu().numpy().T
    err = np.abs(d - ref).max(axis=1)
    assert np.all(err <= tol), err
    assert np.array_equal(d[:4], _eval(gpu, chi))


def test_negative_chi_stays_in_the_table(gpu):
    """Steps too coarse for the field drive the energy through zero, and chi of the
    next stages below it by any amount: such chi takes the last cell (or cell 0
    where it rounds to 0), by itself and in every pass with FP64 steps, and the
    next call on the context gives what it gave before."""
    import torch
    from paper_2308_09348_amd import _lib
    chi = np.concatenate([-2.0 ** np.arange(-60.0, 9.0), [-0.0]])
    assert np.isfinite(_eval(gpu, chi)).all()
    d = gpu.radiation_derivs(torch.tensor(chi, device="cuda"), "fp64").cpu().numpy()
    assert np.isfinite(d).all()
    good = dict(workloads.quantum_batch(n_shots=1)[0], n_samples=700, n_steps=256)
    for precision, chi64 in (("fp64", 0.0), ("fp32", 0.1)):
        q = dict(good, precision=precision, chi_fp64=chi64)
        p = dict(q, n_steps=16)
        ref = gpu.forward(q)["energy_hist"].clone()
        for run in (lambda: gpu.forward(p, check=False),
                    lambda: gpu.forward(p, tape=gpu.new_tape(p["n_samples"]), check=False),
                    lambda: gpu.photons(p, check=False, angles=True)):
            print("negative chi:", precision, chi64, flush=True)
            status = run()["status"].item()
            assert status in (_lib.QS_OK, _lib.QS_ENONFINITE, _lib.QS_ERANGE)
            assert torch.equal(gpu.forward(q)["energy_hist"], ref)
