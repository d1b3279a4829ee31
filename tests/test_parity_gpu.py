"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the
same seeded inputs.

Tolerances for FP64 (stated):
  * the estimate within 1e-10 * max(|ref|, 1);
  * every per-probe quadrature value s_j, and the per-shift means, within
    1e-10 * max(|ref|, 1) of the oracle's;
  * alpha/beta within 1e-8 * max|alpha| (diagnostics only).
Two correct implementations of Algorithm 1 that differ only in rounding
(summation order, the fused Gram-Schmidt pass) agree to about 1e-13 at the
workloads' k; once Ritz values converge next to 0 the quadrature and the late
coefficients become ill-conditioned (measured on the CPU for the 30x30
problem at k = 40: per-probe s_j move by up to 2e-8 = 2e-11 |v|^2 and late
alpha/beta by 1.6e-7 under 1e-16 perturbations of the operator).  The k = 40
cases on that problem therefore bound s_j by 1e-10 * |v_j|^2 (s_j lies in
[0, |v_j|^2], a sum of Gauss weights times |v_j|^2) and alpha/beta by 1e-6.
"""
import json
import math
import os

import numpy as np
import pytest

import oracle
from paper_1602_02306_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")
TOL = 1e-10


@pytest.fixture(scope="module")
def ec():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1602_02306_amd import ecount
    ecount.load()
    return ecount


def gpu_count(ec, A, prec, xi, eta, V, k, **kw):
    Ad = ec.upload_csr(A, val_dtype=kw.pop("val", "f64"))
    vec = kw.get("vec", "f64")
    Vd = torch.from_numpy(V).to("cuda", torch.float32 if vec == "f32" else torch.float64)
    return ec.count(Ad, prec, xi, eta, Vd, k, **kw)


def rel(a, b):
    return abs(a - b) / max(1.0, abs(b))


def assert_parity(r, ref, k=None, coef_tol=1e-8, probe_scale="rel"):
    """probe_scale 'rel': s_j within TOL * max(|s_j|, 1); 'nu': within
    TOL * |v_j|^2 (the ill-conditioned k = 40 cases only, see the header)."""
    s = r.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    nu = np.concatenate([ref.lan_xi.nu, ref.lan_eta.nu])
    scale = np.maximum(1.0, np.abs(s_ref)) if probe_scale == "rel" else nu
    print("gpu %.15f oracle %.15f | rel est %.2e | max |ds|/nu %.2e | max |ds|/max(|s|,1) %.2e"
          % (r.estimate, ref.estimate, rel(r.estimate, ref.estimate),
             np.max(np.abs(s - s_ref) / nu), np.max(np.abs(s - s_ref) / np.maximum(1, np.abs(s_ref)))),
          flush=True)
    assert rel(r.estimate, ref.estimate) <= TOL
    if probe_scale == "rel":
        assert abs(r.neg_xi - ref.neg_xi) <= TOL * max(1.0, abs(ref.neg_xi))
        assert abs(r.neg_eta - ref.neg_eta) <= TOL * max(1.0, abs(ref.neg_eta))
    else:
        nu_mean = float(np.mean(nu))
        assert abs(r.neg_xi - ref.neg_xi) <= TOL * nu_mean
        assert abs(r.neg_eta - ref.neg_eta) <= TOL * nu_mean
    assert np.all(np.abs(s - s_ref) <= TOL * scale)
    if not math.isnan(ref.variance):
        assert abs(r.variance - ref.variance) <= 1e-8 * max(ref.variance, 1e-12)
    ku = r.k_used.cpu().numpy()
    ku_ref = np.concatenate([ref.lan_xi.k_used, ref.lan_eta.k_used])
    assert np.array_equal(ku, ku_ref)
    if k is not None:
        al = r.alpha.cpu().numpy().T
        be = r.beta.cpu().numpy().T
        al_ref = np.concatenate([ref.lan_xi.alpha, ref.lan_eta.alpha])
        be_ref = np.concatenate([ref.lan_xi.beta, ref.lan_eta.beta])
        scale = max(1.0, np.abs(al_ref).max())
        print("max |d alpha| %.2e  max |d beta| %.2e" % (
            max(np.max(np.abs(al[c, :ku_ref[c]] - al_ref[c, :ku_ref[c]])) for c in range(al.shape[0])),
            max(np.max(np.abs(be[c, :ku_ref[c] + 1] - be_ref[c, :ku_ref[c] + 1])) for c in range(al.shape[0]))),
            flush=True)
        for c in range(al.shape[0]):
            kk = ku_ref[c]
            assert np.all(np.abs(al[c, :kk] - al_ref[c, :kk]) <= coef_tol * scale)
            assert np.all(np.abs(be[c, :kk + 1] - be_ref[c, :kk + 1]) <= coef_tol * scale)


def run_workload(ec, name, **over):
    wl = W.WORKLOADS[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    k = over.pop("k", wl.k)
    rule = over.pop("rule", "gauss")
    sw = over.pop("smooth_w", wl.smooth_w)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, k, rule=rule, smooth_w=sw, **over)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, k, rule=rule, smooth_w=sw)
    return r, ref, k


@pytest.mark.parametrize("name", ["c1", "c2_small", "c2_ragged"])
def test_parity_small_workloads(ec, name):
    print("case", name, flush=True)
    r, ref, k = run_workload(ec, name)
    assert_parity(r, ref, k)


def test_parity_ga_rule(ec):
    r, ref, k = run_workload(ec, "c1", rule="ga")
    assert_parity(r, ref, k)


def test_parity_ga_rule_cheb(ec):
    r, ref, k = run_workload(ec, "c2_ragged", rule="ga")
    assert_parity(r, ref, k)


def test_parity_smoothed(ec):
    r, ref, k = run_workload(ec, "c2_small", smooth_w=0.05)
    assert_parity(r, ref, k)


def test_parity_more_than_one_basis_chunk(ec):
    # k = 40 > 32: the reorthogonalization runs over two basis chunks
    r, ref, k = run_workload(ec, "c1", k=40)
    assert_parity(r, ref, k, coef_tol=1e-6, probe_scale="nu")


@pytest.mark.parametrize("prec", ["none", "jacobi", "cheb"])
def test_full_krylov_exact_count_gpu(ec, prec):
    """k = n with Hadamard probes: the estimate is the exact integer count
    (Proposition 1 and eq. negi_T), for every preconditioner."""
    dims = (4, 4, 4)
    wl = W.Workload("t", dims, "wells", 3, -5.0, 1.0, prec, 64, 64)
    P = W.make_problem(wl)
    lam = np.linalg.eigvalsh(P.A.to_dense())
    xi, eta = 0.5 * (lam[5] + lam[6]), 0.5 * (lam[40] + lam[41])
    V = W.hadamard_probes(64)
    r = gpu_count(ec, P.A, P.prec, xi, eta, V, 64)
    assert abs(r.estimate - 35.0) < 1e-9
    ref = oracle.count(P.A, P.prec, xi, eta, V, 64)
    assert rel(r.estimate, ref.estimate) <= TOL


FORMS = {"fused": {}, "waves": {"fused": "off"}}


@pytest.mark.parametrize("form", list(FORMS))
def test_ideal_preconditioner_breakdown_gpu(ec, form):
    """Diagonal A with |A - tau I|^(-1/2): two distinct eigenvalues of C, the
    Lanczos run stops after 2 steps and s_j equals the count (Section 6).
    Both the one-launch form of small problems and the column waves."""
    rng = np.random.default_rng(5)
    d = rng.uniform(-3.0, 3.0, 300)
    A = W.CSR(300, np.arange(301, dtype=np.int32), np.arange(300, dtype=np.int32), d)
    V = W.rademacher(300, 70, 11)
    r = gpu_count(ec, A, W.PrecSpec("jacobi", ()), -0.5, 0.7, V, 6, tune=FORMS[form])
    ku = r.k_used.cpu().numpy()
    assert np.all(ku == 2)
    s = r.per_probe.cpu().numpy()
    assert np.allclose(s[:70], np.sum(d < -0.5), atol=1e-9)
    assert np.allclose(s[70:], np.sum(d < 0.7), atol=1e-9)
    assert abs(r.estimate - np.sum((d >= -0.5) & (d < 0.7))) < 1e-9


@pytest.mark.parametrize("form", list(FORMS))
def test_breakdown_mixed_within_a_wave(ec, form):
    """Diagonal A without preconditioner: probes that are unit vectors span an
    invariant space at once (k_used = 1), a probe on two coordinates after two
    steps, Rademacher probes run to k; all in one wave, each column against the
    oracle (its k_used and s_j) while the others keep iterating.  Both the
    one-launch form of small problems and the column waves."""
    rng = np.random.default_rng(8)
    n = 300
    d = np.sort(rng.uniform(-3.0, 3.0, n))
    A = W.CSR(n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), d)
    V = W.rademacher(n, 6, 21)
    V[:, 0] = 0.0
    V[7, 0] = 1.0
    V[:, 3] = 0.0
    V[200, 3] = 1.0
    V[:, 4] = 0.0
    V[10, 4] = 1.0
    V[250, 4] = -1.0
    print("mixed breakdown", form, flush=True)
    r = gpu_count(ec, A, W.PrecSpec("none", ()), -0.5, 0.7, V, 12, tune=FORMS[form])
    ref = oracle.count(A, W.PrecSpec("none", ()), -0.5, 0.7, V, 12)
    ku = np.concatenate([ref.lan_xi.k_used, ref.lan_eta.k_used])
    assert set(ku.tolist()) >= {1, 2, 12}
    assert_parity(r, ref)


def test_single_probe_variance_nan(ec):
    wl = W.WORKLOADS["c1"]
    P = W.make_problem(wl)
    V = W.rademacher(P.A.n, 1, 5)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, 7)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, 7)
    assert math.isnan(r.variance) and math.isnan(ref.variance)
    assert rel(r.estimate, ref.estimate) <= TOL


def max_k_problem():
    wl = W.Workload("t", (10, 8, 8), "wells", 3, -5.0, 1.0, "cheb", 4, 512)
    P = W.make_problem(wl)
    lam = np.sort(np.linalg.eigvalsh(P.A.to_dense()))
    return P, 0.5 * (lam[40] + lam[41]), 0.5 * (lam[300] + lam[301])


@pytest.mark.parametrize("rule,k", [("gauss", 512), ("ga", 256)])
def test_parity_maximum_k(ec, rule, k):
    """The largest k the library takes (512 for the Gauss rule, 256 for the
    GA rule) on n = 640: a 513-slot basis and the largest tridiagonal
    eigenproblem.  Two FP64 oracles that differ only in rounding order (the C
    oracle and the block oracle at P = 1) agree to 1e-14 |v|^2 here."""
    P, xi, eta = max_k_problem()
    V = W.rademacher(P.A.n, 4, 17)
    print("maximum k", rule, k, flush=True)
    r = gpu_count(ec, P.A, P.prec, xi, eta, V, k, rule=rule)
    ref = oracle.count(P.A, P.prec, xi, eta, V, k, rule=rule)
    assert np.all(ref.lan_xi.k_used == k) and np.all(ref.lan_eta.k_used == k)
    assert_parity(r, ref)


def test_one_step(ec):
    r, ref, k = run_workload(ec, "c2_ragged", k=1)
    assert_parity(r, ref, k)


def test_negcounts_four_shifts(ec):
    """Spectrum slicing: 4 shifts, 3 contiguous intervals in one call."""
    wl = W.WORKLOADS["c2_ragged"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    taus = np.array([-70.0, -55.0, -41.0, -30.0])
    Ad = ec.upload_csr(P.A)
    Vd = torch.from_numpy(V).cuda()
    r = ec.negcounts(Ad, P.prec, taus, Vd, wl.k)
    s_gpu = r.per_probe.cpu().numpy().reshape(4, -1)
    for i, tau in enumerate(taus):
        mean, s, _, _ = oracle.negcount(P.A, P.prec, tau, V, wl.k)
        assert rel(r.negcounts[i], mean) <= TOL
        assert np.all(np.abs(s_gpu[i] - s) <= TOL * np.maximum(1.0, np.abs(s)))
    for t in range(3):
        d = s_gpu[t + 1] - s_gpu[t]
        assert rel(r.counts[t], d.mean()) <= 1e-12


def test_jacobi_singular_reported(ec):
    d = np.array([1.0, 0.5, 3.0, -1.0] * 16)
    A = W.CSR(64, np.arange(65, dtype=np.int32), np.arange(64, dtype=np.int32), d)
    V = W.rademacher(64, 3, 1)
    with pytest.raises(ec.EcntError) as e:
        gpu_count(ec, A, W.PrecSpec("jacobi", ()), 0.5, 2.0, V, 3)
    assert e.value.status == ec.ECNT_ENOTHPD


def test_deterministic_bitwise(ec):
    wl = W.WORKLOADS["c2_small"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    a = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    b = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    assert a.estimate == b.estimate and a.variance == b.variance
    assert torch.equal(a.per_probe, b.per_probe)


def test_bench_configuration_sampled(ec):
    """The benchmark workload at full size (64^3 wells, Chebyshev M, 256
    probes, k = 30), in the launch configuration the benchmark times; the
    oracle recomputes a sample of probes one by one (each probe's Lanczos run
    is independent, so a column subset reproduces its s_j exactly)."""
    wl = W.WORKLOADS["c2"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    print("case c2 full", flush=True)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    s = r.per_probe.cpu().numpy().reshape(2, -1)
    sample = [0, 101, 255]
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V[:, sample], wl.k)
    for t, (sx, se) in enumerate(zip(ref.s_xi, ref.s_eta)):
        j = sample[t]
        assert abs(s[0, j] - sx) <= TOL * max(1.0, abs(sx))
        assert abs(s[1, j] - se) <= TOL * max(1.0, abs(se))
    # whole-run properties: estimate is the mean of the per-probe differences
    d = s[1] - s[0]
    assert rel(r.estimate, d.mean()) <= 1e-12
    exact = json.load(open(os.path.join(GOLDEN, "exact_counts.json"))).get("c2", {}).get("count")
    print("c2 estimate %.4f +- %.4f exact %s" % (r.estimate, math.sqrt(r.variance), exact), flush=True)


def test_bench_configuration_sampled_fp32(ec):
    """The benchmark workload at full size in the FP32 storage form (the
    launch configuration of its bench line): sampled probes against the FP64
    oracle and the estimate against the FP64 path, within the FP32 bound."""
    wl = W.WORKLOADS["c2"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    print("case c2 full fp32", flush=True)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec="f32", val="f32")
    s = r.per_probe.cpu().numpy().reshape(2, -1)
    sample = [3, 128]
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V[:, sample], wl.k)
    nu = float(P.A.n)   # |v_j|^2 of a Rademacher probe
    for t, (sx, se) in enumerate(zip(ref.s_xi, ref.s_eta)):
        j = sample[t]
        print("probe %d: fp32 %.6f %.6f oracle %.6f %.6f" % (j, s[0, j], s[1, j], sx, se), flush=True)
        assert abs(s[0, j] - sx) <= FP32_BOUND * nu
        assert abs(s[1, j] - se) <= FP32_BOUND * nu
    r64 = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    print("estimate fp32 %.8f fp64 %.8f" % (r.estimate, r64.estimate), flush=True)
    assert rel(r.estimate, r64.estimate) <= FP32_BOUND


@pytest.mark.parametrize("name", ["c2_small", "c2_ragged"])
def test_parity_clenshaw_evaluation(ec, name):
    """M evaluated by Clenshaw's recurrence instead of the product of its
    quadratic factors: same polynomial, same parity bar."""
    r, ref, k = run_workload(ec, name, eval="clenshaw")
    assert_parity(r, ref, k)


@pytest.mark.parametrize("max_cols", [30, 37, 1])
def test_parity_column_waves(ec, max_cols):
    """Columns run in waves of at most max_cols (ragged last wave; odd widths
    take the one-column-per-lane kernels); results equal the oracle's."""
    r, ref, k = run_workload(ec, "c2_ragged", max_cols=max_cols)
    assert_parity(r, ref, k)


def test_parity_column_waves_two_basis_chunks(ec):
    """k = 40 (two basis chunks per pass, alpha_i from the second) in column
    waves of 30 (a ragged last wave): every wave against the oracle."""
    r, ref, k = run_workload(ec, "c1", k=40, max_cols=30)
    assert_parity(r, ref, k, coef_tol=1e-6, probe_scale="nu")


@pytest.mark.parametrize("vec", ["f64", "f32"])
def test_parity_padded_slots_in_waves(ec, vec):
    """A block vector of 4096 rows x 32 columns is a power of two in bytes, so
    the basis slots are padded; two waves of 32 columns (m = 32, both shifts)."""
    wl = W.WORKLOADS["c2_small"]
    P = W.make_problem(wl)
    V = W.rademacher(P.A.n, 32, 17)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec=vec, max_cols=32)
    if vec == "f64":
        assert_parity(r, ref, wl.k)
    else:
        s = r.per_probe.cpu().numpy()
        s_ref = np.concatenate([ref.s_xi, ref.s_eta])
        assert abs(r.estimate - ref.estimate) <= 1e-4 * max(1.0, abs(ref.estimate))
        assert np.max(np.abs(s - s_ref)) <= 1e-4 * P.A.n


def test_parity_column_waves_jacobi(ec):
    r, ref, k = run_workload(ec, "c1", max_cols=48)
    assert_parity(r, ref, k)


@pytest.mark.parametrize("tune", [{"tile": "2x4"}, {"tile": "1x8"}, {"tile": "4x4"},
                                  {"tile": "4x4-unfused"}, {"tile": "8x8-wg"},
                                  {"red_waves": 64}, {"red_waves": 65536}, {"csr_vw": 1},
                                  {"tile": "2x4", "red_waves": 8192, "csr_vw": 1}])
def test_parity_launch_shapes(ec, tune):
    """Every launch shape the autotuner may pick gives the oracle's results."""
    r, ref, k = run_workload(ec, "c2_ragged", tune=tune)
    assert_parity(r, ref, k)
    r, ref, k = run_workload(ec, "c2_small", tune=tune)
    assert_parity(r, ref, k)


@pytest.mark.parametrize("m", [1, 32, 33, 64, 65, 96, 97, 128])
def test_fp32_columns_per_lane_edges(ec, m):
    """FP32 count at the widths where the columns per lane change (2 m columns:
    one, two, three and four groups of 64, full and ragged): the grid sweeps
    against the oracle, and every width of the CSR sweep the same bits as the
    default's, each column being summed in the same order."""
    wl = W.WORKLOADS["c2_ragged"]
    P = W.make_problem(wl)
    V = W.rademacher(P.A.n, m, 23)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec="f32")
    s = r.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    assert np.max(np.abs(s - s_ref)) <= 1e-4 * P.A.n
    wl = W.WORKLOADS["c1"]
    P = W.make_problem(wl)
    V = W.rademacher(P.A.n, m, 29)
    outs = [gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, 10, vec="f32", tune={"a_form": "csr", "csr_vw": vw})
            for vw in (0, 1, 2, 4)]
    for o in outs[1:]:
        assert torch.equal(o.per_probe, outs[0].per_probe)


def test_stencil_tile_shapes_bitwise(ec):
    """The plain stencil sweep computes each grid point the same way whatever
    the line block, so the tile shape alone changes no bit of the result."""
    wl = W.WORKLOADS["c2_ragged"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    outs = [gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, tune={"tile": t})
            for t in ("4x4-unfused", "2x4", "1x8")]
    for o in outs[1:]:
        assert o.estimate == outs[0].estimate
        assert torch.equal(o.per_probe, outs[0].per_probe)


@pytest.mark.parametrize("tile", ["4x4", "8x8-wg"])
@pytest.mark.parametrize("name", ["c2_small", "c2_ragged"])
def test_fused_quadratic_sweep_matches_two_sweeps(ec, name, tile):
    """Each quadratic factor of the preconditioner in one fused sweep against
    the same factor as two plain sweeps: the same values up to rounding (the
    fused form sums in the same order; only FMA contraction may differ)."""
    wl = W.WORKLOADS[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    a = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, tune={"tile": tile})
    b = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, tune={"tile": "4x4-unfused"})
    nu = float(P.A.n)
    assert abs(a.estimate - b.estimate) <= 1e-12 * max(1.0, abs(b.estimate))
    assert float((a.per_probe - b.per_probe).abs().max()) <= 1e-12 * nu


@pytest.mark.parametrize("dims,m", [((8, 8, 1), 3), ((5, 17, 2), 33), ((9, 10, 67), 5), ((16, 9, 33), 32),
                                    ((24, 24, 64), 64)])
@pytest.mark.parametrize("vec", ["f64", "f32"])
def test_fused_quadratic_sweep_z_chunks(ec, dims, m, vec):
    """The workgroup sweep splits the z range when its line blocks alone leave
    CUs idle: one to many chunks, ragged last ones, against two plain sweeps.
    FP64: the rounding of a few steps; FP32: its stated bound."""
    wl = W.Workload("z", dims, "wells", 3, -8.0, -2.0, "cheb", m, 4)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    a = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec=vec, val=vec, tune={"tile": "8x8-wg"})
    b = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec=vec, val=vec, tune={"tile": "4x4-unfused"})
    tol = 1e-12 if vec == "f64" else FP32_BOUND
    assert float((a.per_probe - b.per_probe).abs().max()) <= tol * P.A.n
    assert float((a.alpha - b.alpha).abs().max()) <= (1e-11 if vec == "f64" else FP32_BOUND) * float(b.alpha.abs().max())


# FP32 storage form: A values, probes, Lanczos vectors and basis in FP32;
# alpha/beta, every dot product and norm and the tridiagonal eigensolve in
# FP64.  Parity with the FP64 oracle is not expected to 1e-10; the stated
# bound is 1e-4 * max(|estimate|, 1) on the estimate and 1e-4 * |v_j|^2 on each
# per-probe value.
FP32_BOUND = 1e-4


@pytest.mark.parametrize("name", ["c2_small", "c2_ragged", "c1"])
def test_fp32_form_within_stated_bound(ec, name):
    wl = W.WORKLOADS[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec="f32", val="f32")
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    s = r.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    nu = np.concatenate([ref.lan_xi.nu, ref.lan_eta.nu])
    e_est = rel(r.estimate, ref.estimate)
    e_probe = float(np.max(np.abs(s - s_ref) / nu))
    print("fp32 %s: est %.10f oracle %.10f rel %.2e  max|ds|/nu %.2e" % (name, r.estimate, ref.estimate, e_est, e_probe), flush=True)
    assert e_est <= FP32_BOUND
    assert e_probe <= FP32_BOUND


@pytest.mark.parametrize("name,max_cols", [("c2_small", 0), ("c2_ragged", 0), ("c2_ragged", 37)])
def test_fp32_workgroup_sweep_within_stated_bound(ec, name, max_cols):
    """The FP32 form with the preconditioner's quadratic factors in the
    workgroup sweep on 8 x 8 line blocks: an even wave width (two columns per
    lane) and an odd one (waves of 37 columns, one per lane), each within the
    FP32 bound of the FP64 oracle."""
    wl = W.WORKLOADS[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    kw = {"max_cols": max_cols} if max_cols else {}
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec="f32", val="f32",
                  tune={"tile": "8x8-wg"}, **kw)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k)
    s = r.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    nu = np.concatenate([ref.lan_xi.nu, ref.lan_eta.nu])
    e_est = rel(r.estimate, ref.estimate)
    e_probe = float(np.max(np.abs(s - s_ref) / nu))
    print("fp32 wg %s/%d: rel %.2e  max|ds|/nu %.2e" % (name, max_cols, e_est, e_probe), flush=True)
    assert e_est <= FP32_BOUND
    assert e_probe <= FP32_BOUND


@pytest.mark.parametrize("prec_kind", ["none", "jacobi"])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_tiny_problems(ec, n, prec_kind):
    """n = 1..3 rows (far below one tile or wavefront), k = n: the Krylov
    space is the whole space, so every s_j is v_j^T h(C) v_j exactly
    (eq. gauss_quad with k = n)."""
    rng = np.random.default_rng(40 + n)
    d = np.sort(rng.uniform(-3.0, 3.0, n)) + np.arange(n)
    e = rng.uniform(0.2, 0.6, max(n - 1, 0))
    T = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
    rows, cols, vals = [], [], []
    for r in range(n):
        for c in range(max(0, r - 1), min(n, r + 2)):
            rows.append(r)
            cols.append(c)
            vals.append(T[r, c])
    rp = np.searchsorted(np.array(rows), np.arange(n + 1)).astype(np.int32)
    A = W.CSR(n, rp, np.array(cols, dtype=np.int32), np.array(vals))
    lam = np.linalg.eigvalsh(T)
    xi = lam[0] - 0.5 if n == 1 else 0.5 * (lam[0] + lam[1])
    eta = lam[-1] + 0.5
    prec = W.PrecSpec(prec_kind, ())
    V = W.rademacher(n, 3, 7 + n)
    print("tiny n=%d %s" % (n, prec_kind), flush=True)
    r = gpu_count(ec, A, prec, xi, eta, V, n)
    ref = oracle.count(A, prec, xi, eta, V, n)
    assert_parity(r, ref)
    s = r.per_probe.cpu().numpy()
    for t, tau in enumerate((xi, eta)):
        Cd = oracle.dense_operator(A, prec, tau)
        ev, U = np.linalg.eigh(0.5 * (Cd + Cd.T))
        Pm = (U * (ev < 0)) @ U.T
        exact = np.einsum("ij,ik,kj->j", V, Pm, V)
        assert np.all(np.abs(s[3 * t:3 * t + 3] - exact) <= 1e-10 * n)


@pytest.mark.parametrize("k", [40, 128])
def test_fp32_form_more_than_one_basis_chunk(ec, k):
    """FP32 storage past one basis chunk (the Gram column with one column per
    lane beyond 24 basis vectors, alpha_i from the launch that holds q_i):
    within the FP32 bound of the FP64 oracle."""
    if k == 40:
        wl = W.WORKLOADS["c2_small"]
        P = W.make_problem(wl)
        V, xi, eta = W.make_probes(wl), wl.xi, wl.eta
    else:
        P, xi, eta = max_k_problem()
        V = W.rademacher(P.A.n, 4, 17)
    r = gpu_count(ec, P.A, P.prec, xi, eta, V, k, vec="f32", val="f32")
    ref = oracle.count(P.A, P.prec, xi, eta, V, k)
    s = r.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    nu = np.concatenate([ref.lan_xi.nu, ref.lan_eta.nu])
    e_est = rel(r.estimate, ref.estimate)
    e_probe = float(np.max(np.abs(s - s_ref) / nu))
    print("fp32 k=%d: est %.10f oracle %.10f rel %.2e  max|ds|/nu %.2e" % (k, r.estimate, ref.estimate, e_est, e_probe), flush=True)
    assert e_est <= FP32_BOUND
    assert e_probe <= FP32_BOUND


# ---------------------------------------------------------------------------
# Differentiated form: gradient of the erf-smoothed count
# ---------------------------------------------------------------------------

GRAD_CASES = {
    "wells6": W.Workload("wells6", (6, 6, 6), "wells", 1, -160.0, -120.0, "cheb", 6, 8),
    "c2_small": W.WORKLOADS["c2_small"],
    "ragged": W.Workload("ragged", (7, 5, 6), "wells", 4, -120.0, -60.0, "cheb", 9, 10),
}


def grad_setup(ec, name, w=0.05):
    wl = GRAD_CASES[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    Ad = ec.upload_csr(P.A)
    Vd = torch.from_numpy(V).cuda()
    return wl, P, V, Ad, Vd


@pytest.mark.parametrize("name", ["wells6", "c2_small", "ragged"])
def test_smooth_gradient_matches_oracle_tangents(ec, name):
    """<dV, u>, d/dxi and d/deta against the oracle's forward-mode tangents
    (Algorithm 1 differentiated in its literal order), relative 1e-8."""
    w = 0.05
    wl, P, V, Ad, Vd = grad_setup(ec, name, w)
    print("case grad", name, flush=True)
    res, ws = ec.smooth_forward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k, smooth_w=w)
    assert rel(res.estimate, ref.estimate) <= TOL
    dV, dxi, deta = ec.smooth_backward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w, workspace=ws)
    dV = dV.cpu().numpy()
    rng = np.random.default_rng(11)
    for t in range(2):
        u = rng.standard_normal(P.A.n)
        _, d_ref = oracle.count_tangent(P.A, P.prec, wl.xi, wl.eta, V, wl.k, u, 0.0, 0.0, w)
        d_gpu = float(np.dot(dV, u))
        print("  <dV,u> gpu %.12e oracle %.12e" % (d_gpu, d_ref), flush=True)
        assert abs(d_gpu - d_ref) <= 1e-8 * max(abs(d_ref), 1e-12 * np.abs(dV).sum())
    _, dxi_ref = oracle.count_tangent(P.A, P.prec, wl.xi, wl.eta, V, wl.k, np.zeros(P.A.n), 1.0, 0.0, w)
    _, deta_ref = oracle.count_tangent(P.A, P.prec, wl.xi, wl.eta, V, wl.k, np.zeros(P.A.n), 0.0, 1.0, w)
    print("  dxi %.12e / %.12e  deta %.12e / %.12e" % (dxi, dxi_ref, deta, deta_ref), flush=True)
    assert abs(dxi - dxi_ref) <= 1e-8 * max(abs(dxi_ref), 1e-10)
    assert abs(deta - deta_ref) <= 1e-8 * max(abs(deta_ref), 1e-10)


def _grad_vs_oracle(ec, P, xi, eta, V, k, w, seed):
    """Forward per probe at 1e-10 * max(|s_j|, 1) and <dV, u>, dxi, deta
    against the oracle's forward-mode tangents at 1e-8 relative."""
    Ad = ec.upload_csr(P.A)
    Vd = torch.from_numpy(V).cuda()
    res, ws = ec.smooth_forward(Ad, P.prec, xi, eta, Vd, k, w, details=True)
    ref = oracle.count(P.A, P.prec, xi, eta, V, k, smooth_w=w)
    s = res.per_probe.cpu().numpy()
    s_ref = np.concatenate([ref.s_xi, ref.s_eta])
    ds = np.max(np.abs(s - s_ref) / np.maximum(1.0, np.abs(s_ref)))
    print("  estimate gpu %.15f oracle %.15f rel %.2e | max |ds|/max(|s|,1) %.2e"
          % (res.estimate, ref.estimate, rel(res.estimate, ref.estimate), ds), flush=True)
    assert rel(res.estimate, ref.estimate) <= TOL
    assert ds <= TOL
    dV, dxi, deta = ec.smooth_backward(Ad, P.prec, xi, eta, Vd, k, w, workspace=ws)
    dV = dV.cpu().numpy()
    u = np.random.default_rng(seed).standard_normal(P.A.n)
    _, d_ref = oracle.count_tangent(P.A, P.prec, xi, eta, V, k, u, 0.0, 0.0, w)
    _, dxi_ref = oracle.count_tangent(P.A, P.prec, xi, eta, V, k, np.zeros(P.A.n), 1.0, 0.0, w)
    _, deta_ref = oracle.count_tangent(P.A, P.prec, xi, eta, V, k, np.zeros(P.A.n), 0.0, 1.0, w)
    d_gpu = float(np.dot(dV, u))
    print("  <dV,u> gpu %.12e oracle %.12e | dxi %.12e / %.12e | deta %.12e / %.12e"
          % (d_gpu, d_ref, dxi, dxi_ref, deta, deta_ref), flush=True)
    assert abs(d_gpu - d_ref) <= 1e-8 * abs(d_ref)
    assert abs(dxi - dxi_ref) <= 1e-8 * max(abs(dxi_ref), 1e-10)
    assert abs(deta - deta_ref) <= 1e-8 * max(abs(deta_ref), 1e-10)


@pytest.mark.parametrize("k", [30, 32])
def test_smooth_gradient_at_largest_k_several_tiles(ec, k):
    """The differentiated form at the workload's k = 30 and at its limit
    k = 32, with 64 probes (128 columns: two 64-column tiles) on the 16^3
    wells problem."""
    wl = W.Workload("g16", (16, 16, 16), "wells", 1, -8.0, -2.0, "cheb", 64, k, smooth_w=0.05)
    P = W.make_problem(wl)
    print("case grad 16^3 m=64 k=%d" % k, flush=True)
    _grad_vs_oracle(ec, P, wl.xi, wl.eta, W.make_probes(wl), k, 0.05, 21)


@pytest.mark.parametrize("m", [1, 33])
@pytest.mark.parametrize("k", [1, 2, 3, 31])
def test_smooth_gradient_smallest_and_ragged(ec, k, m):
    """The reverse kernels at their edges: orders 1 to 31 of the tridiagonal
    adjoint, one and two column tiles (the last one ragged), 210 rows (chunks
    that are no multiple of four rows).  A wide step keeps every derivative far
    from zero; the tolerances are those of the other gradient tests."""
    wl = W.Workload("g", (5, 6, 7), "wells", 2, -8.0, -2.0, "cheb", m, k, smooth_w=0.5)
    P = W.make_problem(wl)
    print("case grad 5x6x7 m=%d k=%d" % (m, k), flush=True)
    _grad_vs_oracle(ec, P, wl.xi, wl.eta, W.make_probes(wl), k, 0.5, 31)


def test_smooth_gradient_hard_shift_k32(ec):
    """k = 32, 128 columns, on the n = 640 problem with xi just above the 41st
    eigenvalue (near the bottom of the spectrum, where a Gram-Schmidt pass
    that took alpha_i from the same vector as the other coefficients loses
    orthogonality fastest)."""
    P, xi, eta = max_k_problem()
    V = W.rademacher(P.A.n, 64, 23)
    print("case grad n=640 hard shift k=32", flush=True)
    _grad_vs_oracle(ec, P, xi, eta, V, 32, 0.05, 22)


def test_smooth_gradient_finite_differences_gpu(ec):
    """Central differences of the GPU's own smoothed estimate."""
    w = 0.05
    wl, P, V, Ad, Vd = grad_setup(ec, "wells6", w)
    _, ws = ec.smooth_forward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w)
    dV, dxi, deta = ec.smooth_backward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w, workspace=ws)
    u = np.random.default_rng(5).standard_normal(P.A.n)
    h = 1e-4

    def est(Vpot, xi, eta):
        A2 = ec.upload_csr(W.laplacian_csr(wl.dims, Vpot))
        return ec.smooth_forward(A2, P.prec, xi, eta, Vd, wl.k, w)[0].estimate

    fd = (est(P.V + h * u, wl.xi, wl.eta) - est(P.V - h * u, wl.xi, wl.eta)) / (2 * h)
    g = float(np.dot(dV.cpu().numpy(), u))
    assert abs(fd - g) <= 1e-6 * abs(g) + 1e-8
    fd = (est(P.V, wl.xi + h, wl.eta) - est(P.V, wl.xi - h, wl.eta)) / (2 * h)
    assert abs(fd - dxi) <= 1e-6 * abs(dxi) + 1e-8
    fd = (est(P.V, wl.xi, wl.eta + h) - est(P.V, wl.xi, wl.eta - h)) / (2 * h)
    assert abs(fd - deta) <= 1e-6 * abs(deta) + 1e-8


def test_smooth_keep_and_recompute_agree(ec):
    w = 0.05
    wl, P, V, Ad, Vd = grad_setup(ec, "c2_small", w)
    res, ws = ec.smooth_forward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w)
    cnt = ec.count(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, smooth_w=w)
    # the differentiated forward is the count's forward (alpha_i first, then
    # the Gram-Schmidt pass): the same kernels, the same estimate
    assert abs(res.estimate - cnt.estimate) <= 1e-15 * abs(cnt.estimate)
    a = ec.smooth_backward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w, g_est=2.0, workspace=ws)
    b = ec.smooth_backward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w, g_est=2.0, ckpt="recompute")
    assert torch.equal(a[0], b[0]) and a[1] == b[1] and a[2] == b[2]
    c = ec.smooth_backward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, w, g_est=1.0, ckpt="recompute")
    assert torch.allclose(a[0], 2.0 * c[0], rtol=1e-14, atol=0)


def test_smooth_autograd_function(ec):
    from paper_1602_02306_amd.autograd import SmoothCount, SmoothProblem
    w = 0.05
    wl = GRAD_CASES["wells6"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    L = W.laplacian_csr(wl.dims)
    pb = SmoothProblem.from_host(L, P.prec, V, wl.k, w)
    Vt = torch.from_numpy(P.V).cuda().requires_grad_(True)
    xi = torch.tensor(wl.xi, dtype=torch.float64, device="cuda", requires_grad=True)
    eta = torch.tensor(wl.eta, dtype=torch.float64, device="cuda", requires_grad=True)
    out = SmoothCount.apply(Vt, xi, eta, pb)
    (3.0 * out).backward()
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, wl.k, smooth_w=w)
    assert rel(out.item(), ref.estimate) <= TOL
    u = np.random.default_rng(2).standard_normal(P.A.n)
    _, d_ref = oracle.count_tangent(P.A, P.prec, wl.xi, wl.eta, V, wl.k, u, 0.0, 0.0, w)
    assert abs(float(np.dot(Vt.grad.cpu().numpy(), u)) - 3.0 * d_ref) <= 1e-8 * abs(3.0 * d_ref)


def test_smooth_rejects_unsupported(ec):
    wl = W.WORKLOADS["c1"]
    P = W.make_problem(wl)
    Ad = ec.upload_csr(P.A)
    Vd = torch.from_numpy(W.make_probes(wl)).cuda()
    with pytest.raises(ec.EcntError) as e:
        ec.smooth_forward(Ad, P.prec, wl.xi, wl.eta, Vd, wl.k, 0.05)   # Jacobi M depends on A
    assert e.value.status == ec.ECNT_EUNSUPPORTED


def _quadrature_matrix(kind, N):
    rng = np.random.default_rng(N)
    if kind == "random":
        return rng.standard_normal(N), 0.1 + rng.random(max(N - 1, 0))
    if kind == "wilkinson":     # pairs of eigenvalues equal to many digits
        return np.abs(np.arange(N) - 0.5 * (N - 1)), np.ones(max(N - 1, 0))
    if kind == "weak":          # two clusters and couplings near the deflation threshold
        return np.where(np.arange(N) % 2 == 0, 1.0, -1.0), np.full(max(N - 1, 0), 1e-9)
    return np.full(N, 2.0), np.ones(max(N - 1, 0))   # "constant": equal diagonal


@pytest.mark.parametrize("kind", ["random", "wilkinson", "weak", "constant"])
@pytest.mark.parametrize("N", [1, 2, 3, 16, 31, 32, 33, 64, 65, 128, 129, 256, 257, 512])
def test_quadrature_of_given_tridiagonal(ec, kind, N):
    """The tridiagonal eigensolve at the edges of its sizes, on matrices with
    clusters and deflation: Lanczos on a tridiagonal A from e_1 returns A itself,
    so s = sum_{theta < 0} z(1)^2 at a shift in a wide gap is known from a dense
    eigensolve.  A backward-stable solve moves it by a few N eps |T| / gap."""
    a, b = _quadrature_matrix(kind, N)
    T = np.diag(a) + np.diag(b, 1) + np.diag(b, -1)
    w, Z = np.linalg.eigh(T)
    gaps = np.diff(np.concatenate([[w[0] - 1.0], w, [w[-1] + 1.0]]))
    at = np.sort(np.argsort(gaps)[-3:])
    taus = np.array([(w[0] - 1.0 if i == 0 else w[i - 1]) + 0.5 * gaps[i] for i in at])
    rp, ci = [0], []
    for r in range(N):
        ci += [c for c in (r - 1, r, r + 1) if 0 <= c < N]
        rp.append(len(ci))
    val = np.array([T[r, c] for r in range(N) for c in ci[rp[r]:rp[r + 1]]])
    A = W.CSR(N, np.array(rp, np.int32), np.array(ci, np.int32), val)
    V = torch.zeros(N, 1, dtype=torch.float64, device="cuda")
    V[0, 0] = 1.0
    if kind == "weak" and N > 128:
        # couplings of 1e-9 of the diagonal amplify the recurrence's rounding by
        # 1e9 a step; past 128 steps its coefficients overflow, which is an error
        with pytest.raises(ec.EcntError) as e:
            ec.negcounts(ec.upload_csr(A), W.PrecSpec("none"), taus, V, N)
        assert e.value.status == ec.ECNT_EDEVICE
        return
    r = ec.negcounts(ec.upload_csr(A), W.PrecSpec("none"), taus, V, N)
    for tau, s, g in zip(taus, r.per_probe.cpu().numpy(), gaps[at]):
        ref = float(np.sum(Z[0, w < tau] ** 2))
        assert abs(s - ref) <= 64 * max(N, 4) * 2.3e-16 * max(np.abs(w - tau).max(), g) / g, (tau, s, ref)


@pytest.mark.parametrize("m", [1025, 3])
def test_quadrature_of_many_columns_and_small_order(ec, m):
    """Order 16, on both sides of the column count where the lane-per-column
    form takes over: the same probes give the same values to rounding."""
    wl = W.Workload("q", (7, 8, 9), "wells", 2, -8.0, -2.0, "none", 1025, 16)
    P = W.make_problem(wl)
    V = W.make_probes(wl)[:, :m]
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, tune={"fused": "off"})
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V[:, :3], wl.k)
    s = r.per_probe.cpu().numpy().reshape(2, m)[:, :3]
    assert np.max(np.abs(s - np.stack([ref.s_xi, ref.s_eta]))) <= TOL * P.A.n


@pytest.mark.parametrize("k", [1, 2, 16, 17, 33, 49, 112, 113])
@pytest.mark.parametrize("prec,m,cols", [("cheb", 3, 0), ("jacobi", 37, 0), ("cheb", 37, 50)])
def test_one_sweep_step_edges(ec, prec, m, cols, k):
    """The one-sweep Lanczos step against the oracle where its split changes:
    one to four wavefronts of at most 28 slots, a wavefront with fewer slots
    than the others, one and two column tiles (the last one ragged), column
    waves, and k = 113, which the two-read form takes.  n = 693: rows that no
    chunk divides.  s_j is within the oracle's rounding times the conditioning
    of the rule, well below 1e-10 |v_j|^2; alpha and beta lose digits once Ritz
    values converge, so they are compared up to k = 33."""
    wl = W.Workload("e", (9, 7, 11), "wells", 5, -8.0, -2.0, prec, m, k)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, k, tune={"fused": "off"}, max_cols=cols)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, k)
    assert_parity(r, ref, k if k <= 33 else None, probe_scale="nu")


@pytest.mark.parametrize("k", [9, 20, 21, 28, 29, 56, 57, 84, 85])
def test_one_sweep_rows_and_slots_edges(ec, k):
    """As above at the sizes where the rows a wavefront takes at a time change
    (four, two, one, at 8 and 20 slots) and where a wavefront is added (28 each)."""
    wl = W.Workload("e", (9, 7, 11), "wells", 5, -8.0, -2.0, "cheb", 37, k)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, k, tune={"fused": "off"})
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, k)
    assert_parity(r, ref, k if k <= 33 else None, probe_scale="nu")


# ---------------------------------------------------------------------------
# A as a grid stencil (a_form auto) against the CSR sweep (a_form csr)
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("name,vec", [("c2_small", "f64"), ("c2_ragged", "f64"), ("c2_ragged", "f32")])
def test_a_stencil_form_equals_csr_form(ec, name, vec):
    """When A is the grid stencil plus a diagonal, the stencil sweep applies it;
    it sums each row as the CSR sweep does, so both forms agree bitwise."""
    wl = W.WORKLOADS[name]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    print("case a-form", name, vec, flush=True)
    ec.profile_enable(True)
    a = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec=vec, val=vec)
    prof = ec.profile_read()
    ec.profile_enable(False)
    b = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, vec=vec, val=vec, tune={"a_form": "csr"})
    assert prof["op_a_stencil"]["bytes"] > 0 and prof["op_csr"]["bytes"] == 0
    assert a.estimate == b.estimate
    assert torch.equal(a.per_probe, b.per_probe)
    assert torch.equal(a.alpha, b.alpha) and torch.equal(a.beta, b.beta)


def _perturbed(A, rng, how):
    """A copy of A (CSR, both triangles) that is not of the stencil form:
    'coef' scales every symmetric off-diagonal pair by its own factor in
    [0.9, 1.1]; 'extra' adds one symmetric pair of long-range entries."""
    import scipy.sparse as sp
    S = A.to_scipy().tocoo()
    r, c, v = S.row.copy(), S.col.copy(), S.data.copy()
    if how == "coef":
        lo, hi = np.minimum(r, c), np.maximum(r, c)
        f = 1.0 + 0.1 * (2.0 * rng.random(A.n * 8) - 1.0)
        key = (lo * 7919 + hi) % f.size
        v = np.where(r != c, v * f[key], v)
    else:
        i, j = 3, A.n - 5
        r = np.concatenate([r, [i, j]])
        c = np.concatenate([c, [j, i]])
        v = np.concatenate([v, [-0.25, -0.25]])
    M = sp.csr_matrix((v, (r, c)), shape=(A.n, A.n))
    M.sort_indices()
    return W.CSR(A.n, M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data.astype(np.float64))


@pytest.mark.parametrize("how", ["coef", "extra"])
def test_a_not_a_stencil_falls_back_to_csr(ec, how):
    """Variable off-diagonal coefficients, or a coupling outside the stencil:
    the device check rejects the stencil form and the CSR sweep applies A
    (parity with the oracle on the perturbed matrix)."""
    wl = W.WORKLOADS["c2_ragged"]
    P = W.make_problem(wl)
    A2 = _perturbed(P.A, np.random.default_rng(3), how)
    V = W.make_probes(wl)
    print("case a-form fallback", how, flush=True)
    ec.profile_enable(True)
    r = gpu_count(ec, A2, P.prec, wl.xi, wl.eta, V, wl.k)
    prof = ec.profile_read()
    ec.profile_enable(False)
    assert prof["op_csr"]["bytes"] > 0 and prof["op_a_stencil"]["bytes"] == 0
    ref = oracle.count(A2, P.prec, wl.xi, wl.eta, V, wl.k)
    assert_parity(r, ref, wl.k)


def test_hbm_probes_plausible(ec):
    """The stream probes report GB/s between a slow and an impossible rate."""
    for kind in ("copy", "read", "update_mix"):
        g = ec.hbm_probe(kind, 1 << 30, reps=3)
        print("probe", kind, g, flush=True)
        assert 500.0 < g < 9000.0


@pytest.mark.parametrize("prec,k,rule", [("jacobi", 20, "gauss"), ("none", 12, "gauss"),
                                         ("jacobi", 30, "ga"), ("jacobi", 64, "gauss")])
def test_fused_small_form_against_oracle_and_waves(ec, prec, k, rule):
    """c1 (900 rows) runs by default in the one-launch form of small problems
    (M = I or Jacobi, FP64 vectors, k <= 64): against the oracle to the stated
    bar, and against the column-wave kernels (opts.fused = 1), which sum in
    another order, to the same bar.  The profile shows which kernels ran."""
    wl = W.WORKLOADS["c1"]
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    pr = P.prec if prec == "jacobi" else W.PrecSpec("none", ())
    print("case fused", prec, k, rule, flush=True)
    ec.profile_enable(True)
    a = gpu_count(ec, P.A, pr, wl.xi, wl.eta, V, k, rule=rule)
    pa = ec.profile_read()
    ec.profile_enable(True)
    b = gpu_count(ec, P.A, pr, wl.xi, wl.eta, V, k, rule=rule, tune={"fused": "off"})
    pb = ec.profile_read()
    ec.profile_enable(False)
    assert pa["lz_fused"]["launches"] == 1 and pa["lz_dots"]["launches"] == 0
    assert pb["lz_fused"]["launches"] == 0 and pb["lz_dots"]["launches"] >= k
    ref = oracle.count(P.A, pr, wl.xi, wl.eta, V, k, rule=rule)
    scale = "nu" if k >= 40 else "rel"
    assert_parity(a, ref, k, probe_scale=scale)
    assert_parity(b, ref, k, probe_scale=scale)
    assert np.array_equal(a.k_used.cpu().numpy(), b.k_used.cpu().numpy())
    sa, sb = a.per_probe.cpu().numpy(), b.per_probe.cpu().numpy()
    bound = TOL * (np.maximum(1.0, np.abs(sb)) if scale == "rel" else
                   np.concatenate([ref.lan_xi.nu, ref.lan_eta.nu]))
    assert np.all(np.abs(sa - sb) <= bound)


@pytest.mark.parametrize("side,fused", [(40, True), (44, False)])
def test_fused_form_lds_limit(ec, side, fused):
    """The one-launch form holds a column's operator, q and w in LDS (at most
    150 KiB: 28 bytes per row and 12 per nonzero): a 40 x 40 five-point
    operator (1600 rows, 136 KiB) runs in it, 44 x 44 (1936 rows, 164 KiB) in
    the column waves.  Both against the oracle, Jacobi, k = 24."""
    rng = np.random.default_rng(side)
    A = W.laplacian_csr((side, side), rng.uniform(0.0, 1.0, side * side))
    prec = W.PrecSpec("jacobi", ())
    V = W.rademacher(A.n, 8, 77)
    print("case fused limit", side, flush=True)
    ec.profile_enable(True)
    r = gpu_count(ec, A, prec, 0.5, 1.5, V, 24)
    prof = ec.profile_read()
    ec.profile_enable(False)
    assert (prof["lz_fused"]["launches"] == 1) == fused
    assert (prof["lz_dots"]["launches"] > 0) == (not fused)
    ref = oracle.count(A, prec, 0.5, 1.5, V, 24)
    assert_parity(r, ref, 24)


@pytest.mark.parametrize("ea,ev", [(340, 0), (420, 0), (-340, 0), (-420, 0), (100, 470), (-100, -470)])
def test_one_sweep_step_far_from_unit_scale(ec, ea, ev):
    """A and the endpoints times 2^ea, the probes times 2^ev: every quantity of
    the recurrence scales by a power of two, so the counts are those of the
    unscaled call times 4^ev as long as |C|^2 and |v|^2 lie in the range of a
    double, and alpha is its alpha times 2^ea."""
    wl = W.Workload("e", (9, 7, 11), "wells", 5, 2.0, 6.0, "none", 5, 20)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    A = W.CSR(P.A.n, P.A.row_ptr, P.A.col_idx, P.A.val * 2.0 ** ea)
    print("case scale", ea, ev, flush=True)
    a = gpu_count(ec, A, P.prec, wl.xi * 2.0 ** ea, wl.eta * 2.0 ** ea, V * 2.0 ** ev, wl.k, tune={"fused": "off"})
    b = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, wl.k, tune={"fused": "off"})
    assert float((a.per_probe / 4.0 ** ev - b.per_probe).abs().max()) <= TOL * float(b.per_probe.abs().max())
    assert float((a.alpha / 2.0 ** ea - b.alpha).abs().max()) <= 1e-8 * float(b.alpha.abs().max())


def weak_chain(N, b=1e-9):
    """A dense symmetric matrix and a start vector whose Lanczos coefficients are
    alpha = 1, -1, 1, ... and couplings of about b: (A, v, alpha)."""
    a = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    T = np.diag(a) + np.diag(np.full(N - 1, b), 1) + np.diag(np.full(N - 1, b), -1)
    G = np.linalg.qr(np.random.default_rng(N).standard_normal((N, N)))[0]
    D = G @ T @ G.T
    D = 0.5 * (D + D.T)
    A = W.CSR(N, np.arange(0, N * N + 1, N, dtype=np.int32), np.tile(np.arange(N, dtype=np.int32), N), D.ravel())
    return A, G[:, :1].copy(), a


def check_weak_chain(r, a, xi):
    """Rounding turns every q_i by about N eps / b = 1e-5 within its +-1 cluster's
    complement, which moves alpha by its square; a lost basis moves it by 2 and
    more from the first steps on.  v lies in the positive cluster to 1e-9.  (A
    column may stop early: the rounding that the couplings amplify can leave a
    remainder below the breakdown bound as the space runs out.)"""
    al = r.alpha.cpu().numpy()
    ku = int(r.k_used[0])
    assert ku >= len(a) - 8
    assert np.max(np.abs(al[:ku, 0] + xi - a[:ku])) <= 1e-6
    assert np.max(np.abs(r.per_probe.cpu().numpy() - [0.0, 1.0])) <= 1e-8


@pytest.mark.parametrize("N", [8, 16, 33, 64])
def test_fused_form_keeps_the_basis_under_weak_couplings(ec, N):
    """Couplings of 1e-9 of the norm, step after step, in the one-launch form: one
    Gram-Schmidt pass a step loses the basis by step 16."""
    A, v, a = weak_chain(N)
    xi, eta = -2.0, 1.5
    print("case weak fused", N, flush=True)
    ec.profile_enable(True)
    r = gpu_count(ec, A, W.PrecSpec("none"), xi, eta, v, N)
    prof = ec.profile_read()
    ec.profile_enable(False)
    assert prof["lz_fused"]["launches"] == 1
    check_weak_chain(r, a, xi)


@pytest.mark.parametrize("k", [112, 113, 120, 128])
def test_one_sweep_step_keeps_the_basis_under_weak_couplings(ec, k):
    """Couplings of 1e-9 of the norm up to the most steps of the one-sweep form
    (four wavefronts up to 112 slots, five from there on)."""
    A, v, a = weak_chain(144)
    xi, eta = -2.0, 1.5
    print("case weak one-sweep", k, flush=True)
    ec.profile_enable(True)
    r = gpu_count(ec, A, W.PrecSpec("none"), xi, eta, v, k)
    prof = ec.profile_read()
    ec.profile_enable(False)
    assert prof["lz_sweep"]["launches"] == k
    check_weak_chain(r, a[:k], xi)


@pytest.mark.parametrize("rule", ["gauss", "ga"])
@pytest.mark.parametrize("k", [114, 117, 121, 126, 127, 128, 129])
def test_one_sweep_step_five_wavefronts(ec, k, rule):
    """The one-sweep step of 113 to 127 slots (23 to 26 in a wavefront, the last
    one with fewer) and the first order past it, as the smaller orders are tested."""
    wl = W.Workload("e", (9, 7, 11), "wells", 5, -8.0, -2.0, "cheb", 37, k)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, k, rule=rule)
    ref = oracle.count(P.A, P.prec, wl.xi, wl.eta, V, k, rule=rule)
    assert_parity(r, ref, None, probe_scale="nu")


@pytest.mark.parametrize("form,k", [("count", 129), ("count", 150), ("smooth", 32), ("smooth", 16), ("grad", 32),
                                    ("grad", 16), ("batch", 130)])
@pytest.mark.parametrize("b", [1e-9, 1e-5])
def test_lost_basis_ends_a_column(ec, form, k, b):
    """The forms that make one Gram-Schmidt pass a step lose the basis under
    couplings of 1e-9 of the norm (alpha off by 2 and far more within 16 steps).
    The column's result is that of the steps before the lost vector, k_used of
    them, as if they had been asked for (coefficients that leave the range of a
    double afterwards are an error, as they were).  Couplings of 1e-5 are answered
    with all steps."""
    N = 160
    A, v, a = weak_chain(N, b)
    Ad, Vd = ec.upload_csr(A), torch.from_numpy(v).cuda()
    M1 = W.PrecSpec("cheb", (N, 1, 1), 1.0, 1.0, 13.0, np.array([1.0]))   # M = 1
    none = W.PrecSpec("none")
    xi, eta = -2.0, 1.5
    print("case lost basis", form, k, b, flush=True)

    def go(k):
        if form == "count":
            return ec.count(Ad, none, xi, eta, Vd, k)
        if form == "smooth":
            return ec.count(Ad, M1, xi, eta, Vd, k, smooth_w=0.5)
        if form == "grad":
            return ec.smooth_forward(Ad, M1, xi, eta, Vd, k, 0.5, details=True)[0]
        return ec.count_batched(Ad, none, [N], np.array([[xi, eta]]), Vd, k, details=True)
    try:
        r = go(k)
    except ec.EcntError as e:
        assert e.status == ec.ECNT_EDEVICE and b == 1e-9 and k > 128
        return
    ku = r.k_used.cpu().numpy().ravel()
    s = r.per_probe.cpu().numpy().ravel()
    if b == 1e-5:
        assert ku.tolist() == [k, k]
    else:
        assert np.all(ku < 16) and np.all(ku >= 2)
    ref = [0.0, 1.0] if form in ("count", "batch") else [0.5 * math.erfc((1.0 - xi) / 0.5), 0.5 * math.erfc((1.0 - eta) / 0.5)]
    assert np.max(np.abs(s - ref)) <= 1e-8
    if form in ("count", "smooth"):
        al = r.alpha.cpu().numpy()
        for c, t in enumerate((xi, eta)):
            assert np.max(np.abs(al[:ku[c], c] + t - a[:ku[c]])) <= 0.1
            assert np.all(al[ku[c]:, c] == 0.0)
    if form == "grad" and b == 1e-9:
        f = ec.smooth_forward(Ad, M1, xi, eta, Vd, k, 0.5)
        dV, dx, de = ec.smooth_backward(Ad, M1, xi, eta, Vd, k, 0.5, workspace=f[1])
        short = int(ku.min())
        f = ec.smooth_forward(Ad, M1, xi, eta, Vd, short, 0.5)
        dV2, dx2, de2 = ec.smooth_backward(Ad, M1, xi, eta, Vd, short, 0.5, workspace=f[1])
        # a lost vector enters with the square of its coupling: the two shifts' columns
        # may end at different steps
        assert float((dV - dV2).abs().max()) <= 1e-6 and abs(dx - dx2) <= 1e-6 and abs(de - de2) <= 1e-6
        assert abs(float(dV.sum()) + dx + de) <= 1e-6      # a common shift of A, xi and eta changes nothing


def test_exhausted_space_is_answered(ec):
    """A Krylov space of at most 18 dimensions asked for all of them, most of them
    exhausted long before (the 2 x 3 x 3 Laplacian): what comes after the last
    direction is rounding, whether or not the breakdown test sees its remainder,
    and the estimate is the oracle's.  (The gradient's conditioning is that of
    1 / beta; it is finite.)"""
    dims = (2, 3, 3)
    A = W.laplacian_csr(dims)
    prec = W.cheb_invsqrt_prec(dims, 1.0, 2)
    Ad = ec.upload_csr(A)
    rng = np.random.default_rng(3)
    for i in range(40):
        V = W.rademacher(A.n, 48, i) * 0.1
        xi, eta = np.sort(rng.uniform(0.5, 13.0, 2))
        print("case exhausted", i, flush=True)
        r, ws = ec.smooth_forward(Ad, prec, xi, eta, torch.from_numpy(V).cuda(), 18, 0.1)
        dV = ec.smooth_backward(Ad, prec, xi, eta, torch.from_numpy(V).cuda(), 18, 0.1, workspace=ws)[0]
        assert abs(r.estimate - oracle.count(A, prec, xi, eta, V, 18, smooth_w=0.1).estimate) <= TOL
        assert bool(torch.isfinite(dV).all())


def test_weak_couplings_in_fp32_storage(ec):
    """FP32 storage: couplings that small are below its breakdown bound, so the
    column stops there, with what it has; couplings above it keep the basis."""
    for b, ku in ((1e-5, 1), (1e-2, 40)):
        A, v, a = weak_chain(160, b)
        r = gpu_count(ec, A, W.PrecSpec("none"), -2.0, 1.5, v, 40, vec="f32")
        print("case fp32", b, r.k_used.tolist(), flush=True)
        assert r.k_used.tolist() == [ku] * 2
        assert np.max(np.abs(r.per_probe.cpu().numpy() - [0.0, 1.0])) <= 1e-4


def _spread_matrix(kind, N):
    """Tridiagonal matrices on whose eigenvectors e_1 is spread out, and the
    smallest coupling."""
    b = np.ones(N - 1)
    if kind == "chain":         # a band of single eigenvalues
        return 0.1 * np.random.default_rng(N).standard_normal(N), b, 1.0
    if kind == "glued":         # copies of one block: clusters of width 1e-6
        b[20::21] = 1e-6
        return np.zeros(N), b, 1e-6
    w = float(kind)             # pairs, weakly coupled: two clusters, e_1 in all of both
    b[1::2] = w
    return np.zeros(N), b, w


@pytest.mark.parametrize("kind", ["chain", "1e-3", "1e-6", "glued"])
@pytest.mark.parametrize("N", [17, 32, 33, 64, 65, 128, 129, 256, 257, 512])
def test_quadrature_weights_inside_clusters(ec, kind, N):
    """The eigensolve's cumulative weights at shifts that split the mass of e_1
    (reference between 0.02 and 0.98, the widest such gaps), clusters and
    deflation included.  Lanczos is backward stable, T = Q^T (A + E) Q with |E| of
    a few N eps |A|, and so is the eigensolve: a weight moves by N eps |A| / gap
    times a small constant.  T itself moves by the turn of its vectors, up to
    N^2 eps / the smallest coupling: the coefficients are those of the matrix."""
    a, b, w = _spread_matrix(kind, N)
    T = np.diag(a) + np.diag(b, 1) + np.diag(b, -1)
    lam, Z = np.linalg.eigh(T)
    cum = np.cumsum(Z[0] ** 2)[:-1]
    gaps = np.where((cum > 0.02) & (cum < 0.98), np.diff(lam), 0.0)
    at = np.sort([i for i in np.argsort(gaps)[-8:] if gaps[i] > 0.0])
    assert len(at) >= 3
    taus = 0.5 * (lam[at] + lam[at + 1])
    rp, ci = [0], []
    for r in range(N):
        ci += [c for c in (r - 1, r, r + 1) if 0 <= c < N]
        rp.append(len(ci))
    val = np.array([T[r, c] for r in range(N) for c in ci[rp[r]:rp[r + 1]]])
    A = W.CSR(N, np.array(rp, np.int32), np.array(ci, np.int32), val)
    V = torch.zeros(N, 1, dtype=torch.float64, device="cuda")
    V[0, 0] = 1.0
    print("case weights", kind, N, flush=True)
    r = ec.negcounts(ec.upload_csr(A), W.PrecSpec("none"), taus, V, N)
    tol = 64 * N * 2.3e-16 * 4.0 / gaps[at]
    s = r.per_probe.cpu().numpy().ravel()
    assert np.all(np.abs(s - cum[at]) <= tol), (s, cum[at], tol)
    r = ec.count(ec.upload_csr(A), W.PrecSpec("none"), float(taus[0]), float(taus[-1]), V, N)
    ku = int(r.k_used[0])
    assert ku == N or kind == "glued"
    coef = N * N * 2.3e-16 / w
    assert np.max(np.abs(r.alpha.cpu().numpy()[:ku, 0] + taus[0] - a[:ku])) <= coef
    assert np.max(np.abs(r.beta.cpu().numpy()[1:ku, 0] - b[:ku - 1])) <= coef


@pytest.mark.parametrize("kind,size", [("outliers", 1e6), ("outliers", 1e10), ("outliers", 1e11),
                                       ("clusters", 1e-7), ("clusters", 1e-11), ("log", 1e-12)])
@pytest.mark.parametrize("fused", ["auto", "off"])
def test_ill_scaled_operators(ec, kind, size, fused):
    """A diagonal matrix, whose products round once, and probes of +-1: with k = n
    s_j is the number of eigenvalues below the shift.  Lanczos returns it for a
    matrix within a few n eps |A|, which turns an eigenvector by that over its gap
    to the other side; both forms that keep the basis, against that bound."""
    n = 64
    if kind == "outliers":
        lam = np.concatenate([np.linspace(-1.0, 1.0, n - 4), size * np.array([1.0, 2.0, -1.0, 3.0])])
    elif kind == "clusters":
        lam = np.repeat(np.linspace(-1.0, 1.0, 16), 4) + size * np.tile(np.arange(4), 16)
    else:
        h = np.logspace(np.log10(size), 0.0, n // 2)
        lam = np.concatenate([-h, h]) + 0.5
    xi, eta = (-0.1, 0.25) if kind != "log" else (0.1, 0.9)
    lam = np.random.default_rng(4).permutation(lam)
    A = W.CSR(n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), lam)
    V = W.rademacher(n, 5, 8)
    print("case ill-scaled", kind, size, fused, flush=True)
    r = gpu_count(ec, A, W.PrecSpec("none"), xi, eta, V, n, tune={"fused": fused})
    gap = min(np.min(lam[lam > t]) - np.max(lam[lam < t]) for t in (xi, eta))
    tol = 4 * n * 2.3e-16 * np.abs(lam).max() / gap + 1e-9
    s = r.per_probe.cpu().numpy().reshape(2, 5)
    assert np.max(np.abs(s[0] - np.sum(lam < xi))) <= tol
    assert np.max(np.abs(s[1] - np.sum(lam < eta))) <= tol


@pytest.mark.parametrize("coef", [[0.4], [0.5, -0.1], [0.5, -0.1, 0.0], [0.5, -0.12, 0.04, -0.02, 0.0]])
@pytest.mark.parametrize("k", [2, 17])
def test_smooth_gradient_of_polynomials_without_product_form(ec, coef, k):
    """Degrees 0 and 1 and a vanishing leading coefficient are applied by
    Clenshaw's recurrence; the reverse sweep adds M u to what is there."""
    dims = (5, 6, 7)
    wl = W.Workload("g", dims, "wells", 2, -8.0, -2.0, "cheb", 9, k, smooth_w=0.5)
    P = W.make_problem(wl)
    P.prec = W.PrecSpec("cheb", dims, 1.0, 1.0, 13.0, np.array(coef))
    print("case grad clenshaw", coef, k, flush=True)
    _grad_vs_oracle(ec, P, -3.0, 1.0, W.make_probes(wl), k, 0.5, 31)


@pytest.mark.parametrize("prec,vec", [("none", "f64"), ("cheb", "f64"), ("jacobi", "f32")])
@pytest.mark.parametrize("fused", ["auto", "off"])
def test_one_step_with_a_probe_that_is_not_finite(ec, prec, vec, fused):
    """k = 1 needs no eigensolve: a probe with an infinite entry makes its own value
    (and the mean) not a number and is no error; the other probes keep theirs."""
    wl = W.Workload("e", (5, 6, 7), "wells", 2, -8.0, -2.0, prec, 6, 1)
    P = W.make_problem(wl)
    V = W.make_probes(wl)
    ok = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, 1, vec=vec, tune={"fused": fused}).per_probe.cpu().numpy()
    V = V.copy()
    V[3, 2] = np.inf
    r = gpu_count(ec, P.A, P.prec, wl.xi, wl.eta, V, 1, vec=vec, tune={"fused": fused})
    s = r.per_probe.cpu().numpy()
    rest = [c for c in range(12) if c % 6 != 2]
    assert np.array_equal(s[rest], ok[rest])
    assert not np.isfinite(s[[2, 8]]).any() and math.isnan(r.estimate)


@pytest.mark.parametrize("entry", [1e300, math.inf, math.nan])
@pytest.mark.parametrize("form,k", [("count", 2), ("count", 9), ("arnoldi", 3)])
def test_overflow_is_an_error_not_a_breakdown(ec, entry, form, k):
    """An entry of A whose square leaves the range of a double: |u|^2 is not finite,
    which is no small remainder, so the count is EDEVICE and not the rule of the
    steps before it."""
    dims = (6, 5, 7)
    A = W.laplacian_csr(dims)
    val = A.val.copy()
    val[40] = entry
    A = W.CSR(A.n, A.row_ptr, A.col_idx, val)
    Ad, V = ec.upload_csr(A), torch.from_numpy(W.rademacher(A.n, 4, 3)).cuda()
    with pytest.raises(ec.EcntError) as e:
        if form == "count":
            ec.count(Ad, W.cheb_invsqrt_prec(dims, 1.0, 4), 2.0, 7.0, V, k)
        else:
            T = W.PrecSpec("cheb", dims, 1.0, 1.0, 13.0, W.cheb_interp_coeffs(lambda x: 1.0 / x, 1.0, 13.0, 8))
            ec.count_arnoldi(Ad, T, 2.0, 7.0, V, k)
    assert e.value.status == ec.ECNT_EDEVICE
