"""The derivative tape: a forward pass that records, per sample, mu_f, sig2_f
and their derivatives along the eight parameters, and the adjoint read from
it.

  - the adjoint from the tape is bit-for-bit the adjoint that integrates the
    trajectories again (same per-sample arithmetic, same reduction order);
  - the tape's per-sample derivatives match the oracle's forward-mode
    derivatives of the same sample (FP64: 1e-8 relative; FP32: 1e-4, with a
    floor of 1e-9 (FP64) / 1e-6 (FP32) of mu_f per unit of the parameter's
    scale for derivatives that are nearly zero);
  - the tape forward's histograms and moments pass the forward parity bar
    against the oracle (they are not bit-identical to qs_forward's: the FP32
    step arithmetic differs);
  - a batched tape holds each shot's single-call tape at the shot's offset.
"""
import numpy as np
import pytest

from paper_2308_09348_amd import workloads

pytestmark = pytest.mark.gpu

NAMES = ["a0", "w0_um", "x_off_um", "y_off_um", "delay_fs", "gamma0", "sigma_gamma", "div_mrad"]
SCALE = {"a0": 1.0, "w0_um": 3.0, "x_off_um": 3.0, "y_off_um": 3.0, "delay_fs": 30.0,
         "gamma0": 1.0, "sigma_gamma": 1.0, "div_mrad": 1.0}


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09348_amd as qs
    ctx = qs.Context(0)
    yield ctx
    ctx.close()


def _case(n_samples=600, n_steps=256, **kw):
    p = workloads.scaled(workloads.differentiation(), n_samples=n_samples, n_steps=n_steps)
    p.update(kw)
    return p


def _weights(n, seed=5):
    import torch
    rng = np.random.Generator(np.random.PCG64(seed))
    return torch.tensor(rng.normal(size=n + 2), dtype=torch.float64, device="cuda")


CONFIGS = [dict(rr_model="quantum", amp_mode="local", deposit="gauss"),
           dict(rr_model="quantum", amp_mode="a0eff", deposit="cic"),
           dict(rr_model="classical", amp_mode="local", deposit="gauss")]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("cfg", range(len(CONFIGS)))
def test_tape_adjoint_equals_recompute(gpu, precision, cfg):
    p = _case(precision=precision, **CONFIGS[cfg])
    tape = gpu.new_tape(p["n_samples"])
    gpu.forward(p, tape=tape)
    w = _weights(p["n_e"])
    a = gpu.backward(p, w, tape=tape).cpu().numpy()
    b = gpu.backward(p, w).cpu().numpy()
    assert np.array_equal(a, b), (a, b)


def _check_sample_derivs(oracle, p, tape, idx, rtol, floor):
    t = tape.cpu().numpy()
    worst = 0.0
    for i in idx:
        m, s2 = oracle.sample_grad(p, int(i))
        assert abs(t[0, i] - m[0]) <= rtol * abs(m[0]), (i, t[0, i], m[0])
        assert abs(t[1, i] - s2[0]) <= rtol * abs(s2[0]) + floor * m[0] ** 2, (i, t[1, i], s2[0])
        for k, name in enumerate(NAMES):
            fl = floor * abs(m[0]) / SCALE[name]
            dm = abs(t[2 + k, i] - m[1 + k])
            ds = abs(t[10 + k, i] - s2[1 + k])
            worst = max(worst, dm / (abs(m[1 + k]) + fl), ds / (abs(s2[1 + k]) + fl * abs(m[0])))
            assert dm <= rtol * abs(m[1 + k]) + fl, (i, name, t[2 + k, i], m[1 + k])
            assert ds <= rtol * abs(s2[1 + k]) + fl * abs(m[0]), (i, name, t[10 + k, i], s2[1 + k])
    return worst


@pytest.mark.parametrize("precision,rtol,floor", [("fp64", 1e-8, 1e-9), ("fp32", 1e-4, 1e-6)])
@pytest.mark.parametrize("cfg", range(len(CONFIGS)))
def test_tape_matches_oracle_sample_derivatives(gpu, oracle, precision, rtol, floor, cfg):
    p = _case(n_samples=300, precision=precision, **CONFIGS[cfg])
    tape = gpu.new_tape(p["n_samples"])
    gpu.forward(p, tape=tape)
    worst = _check_sample_derivs(oracle, p, tape, range(0, 300, 23), rtol, floor)
    print(precision, CONFIGS[cfg], "worst relative", worst)


def test_tape_forward_parity_with_oracle(gpu, oracle):
    p = _case(n_samples=3000, n_steps=512, deposit="cic")
    g = gpu.forward(p, tape=gpu.new_tape(p["n_samples"]))
    g = {k: v.cpu().numpy() for k, v in g.items()}
    o = oracle.forward(p)
    assert g["moments"][0] == p["n_samples"]
    for m in (1, 2, 4, 6, 7, 9, 10):
        assert abs(g["moments"][m] - o["moments"][m]) <= 1e-5 * abs(o["moments"][m]), m
    assert abs(g["moments"][8] - o["moments"][8]) <= 1e-5 * o["moments"][8]
    for key in ("energy_hist", "angle_hist"):
        tol = 1e-4 * o[key] + 1e-7 * o[key].sum()
        assert np.all(np.abs(g[key] - o[key]) <= tol), key
    assert np.array_equal(g["a0eff_hist"], o["a0eff_hist"])


def test_full_size_sampled(gpu, oracle):
    """The differentiation workload at its full size (2^20 samples x 1024
    steps, FP32, the launch the benchmark times): sampled tape entries
    against the oracle's per-sample derivatives, and the gradient's
    consistency between tape and recompute."""
    p = workloads.differentiation()
    n = p["n_samples"]
    tape = gpu.new_tape(n)
    out = gpu.forward(p, tape=tape)
    assert out["energy_hist"].sum().item() == n
    idx = np.linspace(0, n - 1, 12).astype(np.int64)
    worst = _check_sample_derivs(oracle, p, tape, idx, 1e-4, 1e-6)
    print("full size worst relative", worst)
    w = _weights(p["n_e"])
    a = gpu.backward(p, w, tape=tape).cpu().numpy()
    b = gpu.backward(p, w).cpu().numpy()
    assert np.array_equal(a, b)


def test_batched_tape_equals_single(gpu):
    import torch
    base = _case(n_samples=300)
    shots = [dict(base, n_samples=n, a0=a0, gamma0=g0, sigma_gamma=0.05 * g0, e_hi=1.5 * g0)
             for n, a0, g0 in [(1, 20.0, 2000.0), (700, 50.0, 1500.0), (2500, 80.0, 3000.0)]]
    total = sum(s["n_samples"] for s in shots)
    tape = gpu.new_tape(total)
    outs = gpu.forward_batched(shots, tape=tape)
    ws = [_weights(s["n_e"], seed=k) for k, s in enumerate(shots)]
    grads = gpu.backward_batched(shots, ws, tape=tape)
    off = 0
    for k, s in enumerate(shots):
        q = dict(s, shot=s["shot"] + k)
        t1 = gpu.new_tape(s["n_samples"])
        o1 = gpu.forward(q, tape=t1)
        assert torch.equal(tape[:, off:off + s["n_samples"]], t1), k
        for key in ("energy_hist", "angle_hist", "a0eff_hist", "moments"):
            assert torch.equal(outs[k][key], o1[key]), (k, key)
        assert torch.equal(grads[k], gpu.backward(q, ws[k], tape=t1)), k
        off += s["n_samples"]


def test_tape_rejects_bad_tensor(gpu):
    import torch
    p = _case(n_samples=100)
    with pytest.raises(ValueError):
        gpu.forward(p, tape=torch.empty((18, 99), dtype=torch.float64, device="cuda"))


@pytest.mark.parametrize("chi_fp64,n_e", [(0.0, 60), (0.0, 4096), (0.1, 60), (0.1, 4096)])
@pytest.mark.parametrize("deposit", ["point", "cic", "gauss"])
def test_contraction_of_given_laws(gpu, deposit, chi_fp64, n_e):
    """The law sensitivities alone: a tape whose derivatives are one (of mu along
    a0, of sig2 along w0) gives the sums of dL/dmu and dL/dsig2, here against
    erfc and exp, for laws from point-like to 50 bins wide, on either side of
    the box law's change of form at a quarter bin (s = 4 bins), in and outside
    the window.  The densities follow by products of at most 16 factors, so
    terms carry up to ~16^2 roundings and the erfc differences n_e 1e-16 of
    theirs: 1e-12 of the sum of magnitudes."""
    import torch
    from scipy.special import erfc
    p = _case(n_samples=2100, n_e=n_e, e_lo=0.0, e_hi=3000.0, deposit=deposit,
              chi_fp64=chi_fp64)
    wb = p["e_hi"] / n_e
    rng = np.random.Generator(np.random.PCG64(3))
    s = wb * np.resize([0.0, 0.05, 0.5, 1.0, 3.999, 4.0, 4.001, 7.3, 20.0, 50.0], 2100)
    mu = rng.uniform(1.0, p["e_hi"] + 20 * wb, 2100)
    tape = gpu.new_tape(2100)
    tape.zero_()
    tape[0] = torch.tensor(mu)
    tape[1] = torch.tensor(s * s)
    tape[2] = 1.0
    tape[2 + 8 + 1] = 1.0
    w = _weights(n_e)
    gpu.forward(p)  # (the tables of this precision)
    g = gpu.backward(p, w, tape=tape).cpu().numpy()

    W = w.cpu().numpy()
    c = np.concatenate([[W[n_e]], W[:n_e]]) - np.concatenate([W[:n_e], [W[n_e + 1]]])
    t = wb * np.arange(n_e + 1)[None] - mu[:, None]
    se = np.hypot(s, p["kernel_sigma_bins"] * wb) if deposit == "gauss" else s
    with np.errstate(divide="ignore", invalid="ignore"):
        dse = np.where(s > 0, 0.5 / se, 0.0)[:, None]
        pdf = lambda x: np.exp(-0.5 * (x / se[:, None]) ** 2) / np.sqrt(2 * np.pi)
        if deposit == "cic":
            a, b = np.abs(t) - 0.5 * wb, np.abs(t) + 0.5 * wb  # (even in t)
            r = se[:, None] * np.sqrt(2.0)
            dv = -0.5 * (erfc(a / r) - erfc(b / r)) / wb
            ds = (pdf(t + 0.5 * wb) - pdf(t - 0.5 * wb)) / wb * dse
            dv = np.where(s[:, None] > 0, dv, np.where(np.abs(t) < 0.5 * wb, -1.0 / wb, 0.0))
        else:
            dv = -pdf(t) / se[:, None]
            ds = -(t / se[:, None]) * pdf(t) / se[:, None] * dse
            if deposit == "point":
                dv = np.where(s[:, None] > 0, dv, 0.0)
        ds = np.where(s[:, None] > 0, ds, 0.0)
    assert abs(g[0] - (c * dv).sum()) <= 1e-12 * np.abs(c * dv).sum()
    assert abs(g[1] - (c * ds).sum()) <= 1e-12 * np.abs(c * ds).sum()
    assert not g[2:].any()


@pytest.mark.parametrize("n_samples,n_steps", [(1, 130), (64, 131), (65, 4), (300, 3), (1111, 5),
                                               (2500, 513), (513, 1)])
def test_small_tape_has_the_bits_of_a_large_one(gpu, n_samples, n_steps):
    """FP32 quantum tape passes of at most an item a CU divide a step over three
    wavefronts; beside a shot of 70,000 samples (274 items) the same shot goes
    through the general kernel.  Counts of steps at and between multiples of the
    four that a buffer holds, samples at the edges of wavefronts and items."""
    import torch
    p = _case(n_samples=n_samples, n_steps=n_steps, a0=3.0 if n_steps < 100 else 30.0)
    big = dict(p, n_samples=70_000)
    t1 = gpu.new_tape(n_samples)
    o1 = gpu.forward(p, tape=t1)
    t2 = gpu.new_tape(n_samples + 70_000)
    o2 = gpu.forward_batched([p, big], tape=t2)[0]
    assert torch.equal(t1, t2[:, :n_samples])
    for key in o1:
        assert torch.equal(o1[key], o2[key]), key


@pytest.mark.parametrize("deposit,n_e,dz,bound_v,bound_s", [
    ("cic", 4096, (0.0032, 0.032), 1.2e-15, 1.5e-15), ("point", 256, (0.032, 0.25), 6.5e-16, 7e-16)])
def test_contraction_rounding(gpu, deposit, n_e, dz, bound_v, bound_s):
    """Derivatives of laws given by the tape (one sample a shot) against extended
    precision, as a share of the sum of magnitudes, rms over 400 laws.  The same
    recurrences on the CPU give 3.1e-16 (centre) and 4.1e-16 (width) for boxes of 0.003
    to 0.03 standard deviations, 4.0e-16 and 5.3e-16 for normal laws; with the box
    ends' densities subtracted 7.3e-15 (width), with sixteen edges a chunk 8.7e-16 and
    9.2e-16 for normal laws."""
    import torch
    n, width = 400, 3072.0 / n_e
    rng = np.random.Generator(np.random.PCG64(8))
    step = np.exp(rng.uniform(np.log(dz[0]), np.log(dz[1]), n))
    mu, s2 = 3072.0 * rng.uniform(0.2, 0.8, n), (width / step) ** 2
    shots = [dict(_case(n_samples=1, n_steps=8), precision="fp64", deposit=deposit, n_e=n_e,
                  e_lo=0.0, e_hi=3072.0) for _ in range(n)]
    tape = np.zeros((18, n))
    tape[0], tape[1] = mu, s2
    tape[2] = 1.0        # the first parameter moves mu
    tape[2 + 8 + 1] = 1.0  # the second sig2
    ph, fr = rng.uniform(0, 6, n), rng.uniform(0, 0.5, n)
    w = np.zeros((n, n_e + 2))
    w[:, :n_e] = np.sin(ph[:, None] + fr[:, None] * np.arange(n_e))
    w[:, n_e], w[:, n_e + 1] = np.sin(ph - fr), np.sin(ph + fr * n_e)
    grads = gpu.backward_batched(shots, [torch.tensor(a, device="cuda") for a in w],
                                 tape=torch.tensor(tape, device="cuda"))
    g = np.array([x.cpu().numpy() for x in grads])
    L = np.longdouble
    e = L(width) * np.arange(n_e + 1)
    x, gw = np.polynomial.legendre.leggauss(12)
    norm = 1 / np.sqrt(2 * np.arccos(L(-1)))
    err = []
    for k in range(n):
        c = L(np.concatenate(([w[k, n_e]], w[k, :n_e])) -
              np.concatenate((w[k, :n_e], [w[k, n_e + 1]])))
        s = np.sqrt(L(s2[k]))
        z, d = (e - L(mu[k])) / s, L(width) / s / 2
        phi = lambda t: norm * np.exp(-t * t / 2)
        if deposit == "cic":
            mass = sum(L(b) * phi(z + d * L(a)) for a, b in zip(x, gw)) * d
            dv, ds = -c * mass / width, c * (phi(z + d) - phi(z - d)) / width / (2 * s)
        else:
            dv, ds = -c * phi(z) / s, -c * z * phi(z) / s / (2 * s)
        err.append([float((g[k, 0] - dv.sum()) / np.abs(dv).sum()),
                    float((g[k, 1] - ds.sum()) / np.abs(ds).sum())])
    rms = np.sqrt(np.mean(np.square(err), axis=0))
    print("centre, width", rms)
    assert rms[0] < bound_v and rms[1] < bound_s
