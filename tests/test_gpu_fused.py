"""The fused, LDS-tiled, k-marching stage kernel against the one-thread-per-
node reference kernel (both GPU) and against the oracle, on sizes chosen to
leave ragged tiles in i and j and chunk boundaries in k; and the
mixed-precision path against the FP64 oracle with its stated error bound."""
import os

import numpy as np
import pytest

from paper_2003_08746_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lesmi():
    import torch
    assert torch.cuda.is_available()
    from paper_2003_08746_amd import lesmi as L
    L.lib()
    return L


def _rel(a, b):
    ai, bi = I.interior(a), I.interior(b)
    den = np.abs(bi).reshape(bi.shape[0], -1).max(1)
    den = np.where(den == 0, 1.0, den)
    return np.abs(ai - bi).reshape(ai.shape[0], -1).max(1) / den


@pytest.mark.parametrize("shape,prec", [((5, 5, 5), 0), ((30, 14, 8), 0), ((31, 15, 33), 0), ((60, 28, 300), 0),
                                        ((200, 100, 21), 0), ((31, 15, 33), 1), ((331, 155, 12), 0),
                                        ((331, 155, 12), 1)])
def test_automatic_schedule_bitwise(lesmi, shape, prec, monkeypatch):
    """The automatic number of k chunks over its range: one plane per segment,
    one tile, a second tile of one row and column, many chunks of one tile,
    several rounds of blocks, and chunks of two sizes (3 and 4 planes of 144
    tiles).  The arithmetic of a point does not depend on
    the schedule, so the result equals that of chunks of 7 planes bit for
    bit."""
    ni, nj, nk = shape
    case = I.jet_case(ni, nj, nk, seed=3)
    print(f"[gpu] automatic schedule {shape} prec={prec}", flush=True)
    monkeypatch.delenv("LES_SEG", raising=False)
    a = lesmi.Solver(case, prec=prec)
    monkeypatch.setenv("LES_SEG", "7")
    b = lesmi.Solver(case, prec=prec)
    Qa, Qb = a.upload(case["Q"]), b.upload(case["Q"])
    a.rk_step(Qa, 1e-3)
    b.rk_step(Qb, 1e-3)
    assert np.array_equal(a.download(Qa), b.download(Qb))
    a.close()
    b.close()


def _ghost_cases():
    n = (5, 6, 7)
    per = I.periodic_case(*n, I.wavy_grid(*n, L=(1.0, 1.2, 1.4), amp=0.2), I.smooth_state(*n, seed=13, amp=0.1),
                          mu_ref=3e-3, sgs=1)
    jet = I.jet_case(61, 29, 23, seed=3)
    return {"periodic5x6x7": per, "jet61x29x23": jet, "jet30x14x5": I.jet_case(30, 14, 5, seed=3),
            "jet61x29x23_dyn": I.jet_case(61, 29, 23, seed=3, sgs=2), "superposed_i": I.superposed_case(jet, 0),
            "superposed_k": I.superposed_case(jet, 2), "ogrid24x16x21": I.ogrid_case(24, 16, 21, seed=2)}


GHOST_CASES = _ghost_cases()


@pytest.mark.parametrize("name", list(GHOST_CASES))
def test_wrapped_ghosts_bitwise(lesmi, name):
    """Steps whose stages read periodic ghosts at their source against steps
    with stage checkpoints, whose ghosts are filled: the same values, so the
    same results bit for bit.  Every ghost of Q is perturbed, so that frozen
    edge ghosts of periodic and Dirichlet directions differ from the values
    at their periodic images."""
    import torch
    case = dict(GHOST_CASES[name])
    rng = np.random.default_rng(41)
    Q = case["Q"] * (1.0 + 1e-3 * rng.uniform(-1, 1, size=case["Q"].shape))
    sl = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    Q[sl] = case["Q"][sl]
    print(f"[gpu] wrapped ghosts {name}", flush=True)
    s = lesmi.Solver(case)
    ck = torch.empty(25 * s.fe, dtype=torch.float64, device="cuda")
    Qa, Qb = s.upload(Q), s.upload(Q)
    for _ in range(2):
        s.rk_step(Qa, 1e-4)
        s.rk_step(Qb, 1e-4, ckpt=ck)
    A, B = s.download(Qa), s.download(Qb)
    assert np.isfinite(I.interior(A)).all() and not np.array_equal(I.interior(A), I.interior(case["Q"]))
    assert np.array_equal(A, B)
    # several steps in one call (no fill between them where nothing needs it)
    Qa, Qb = s.upload(Q), s.upload(Q)
    dts, _ = s.advance(Qa, 3, want_dt=True)
    for dt in dts:
        s.rk_step(Qb, float(dt), ckpt=ck)
    assert np.array_equal(s.download(Qa), s.download(Qb))
    s.close()


def _filled_cases():
    out = {k: (c, None) for k, c in GHOST_CASES.items()}
    out["ogrid24x16x21_dyn"] = (I.ogrid_case(24, 16, 21, seed=2, sgs=2), None)
    out["superposed_i_dyn"] = (I.superposed_case(I.jet_case(61, 29, 23, seed=3, sgs=2), 0), None)
    # i Dirichlet (entrance, exit) and j Dirichlet (far field), k periodic or
    # superposed; and with the j-hi far field of the O-grid
    jet = I.jet_case(61, 29, 23, seed=3)
    out["faces_k_periodic"] = (dict(jet, bc=(1, 1, 0)), (1, 2, 3, 3))
    out["faces_k_superposed"] = (dict(I.superposed_case(jet, 2), bc=(1, 1, 2)), (1, 2, 3, 0))
    out["faces_i_periodic"] = (jet, (0, 0, 3, 3))
    out["faces_ogrid"] = (I.ogrid_case(24, 16, 21, seed=2), (0, 0, 0, 3))
    return out


FILLED_CASES = _filled_cases()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", list(FILLED_CASES))
def test_steps_against_filled_ghosts(lesmi, name, prec):
    """Steps that read periodic ghosts at their source and keep frozen ghosts in
    the stage buffers against steps with every ghost filled before every stage,
    in both precisions, with boundary faces and with the dynamic closure: the
    same values, so the same results bit for bit.  Every ghost is perturbed, as
    above."""
    base, faces = FILLED_CASES[name]
    case = dict(base)
    rng = np.random.default_rng(43)
    Q = case["Q"] * (1.0 + 1e-3 * rng.uniform(-1, 1, size=case["Q"].shape))
    sl = (slice(None), slice(2, -2), slice(2, -2), slice(2, -2))
    Q[sl] = case["Q"][sl]
    print(f"[gpu] steps against filled ghosts {name} prec={prec}", flush=True)
    s = lesmi.Solver(case, prec=prec)
    if faces:
        outside = s.upload(I.outside_state(case, cross=(0.0, 0.0, 0.03)))
        for f, t in enumerate(faces):
            if t:
                s.set_face(f, t, outside, p_exit=1.0 / I.GAMMA if t == 2 else 0.0)
    got = []
    for on in (False, True):
        lesmi.les_debug_fill_ghosts(s.ctx, on)
        q = s.upload(Q)
        step = s.rk_step(q, 0.0, want_dt=True, want_norms=True)
        adv = s.advance(q, 4, want_dt=True, want_norms=True)
        got.append((s.download(q), step[0], step[1], adv[0], adv[1]))
    assert np.isfinite(I.interior(got[0][0])).all() and not np.array_equal(I.interior(got[0][0]), I.interior(Q))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    s.close()


def _metric_copy_cases():
    n = (31, 15, 9)
    wavy = I.wavy_grid(*n, L=(2.0, 1.5, 1.0), amp=0.2)
    return {"jet61x29x23": I.jet_case(61, 29, 23, seed=3), "jet61x29x23_dyn": I.jet_case(61, 29, 23, seed=3, sgs=2),
            "wavy_ci": I.periodic_case(*n, wavy, I.smooth_state(*n, seed=7, amp=0.1), mu_ref=3e-3, sgs=1, CI=0.05),
            "wavy_alpha07": I.periodic_case(*n, wavy, I.smooth_state(*n, seed=7, amp=0.1), mu_ref=3e-3, alpha=0.7),
            "ogrid24x16x21": I.ogrid_case(24, 16, 21, seed=2),
            "ogrid24x16x21_dyn": I.ogrid_case(24, 16, 21, seed=2, sgs=2)}


METRIC_COPY_CASES = _metric_copy_cases()


@pytest.mark.parametrize("name", list(METRIC_COPY_CASES))
def test_mixed_without_metric_copy_bitwise(lesmi, name):
    """Mixed steps that take their metric terms from the FP64 fields (a context
    without memory for the FP32 copy) against steps that take them from the
    copy, in every instantiation of the stage kernel: the same FP32 values, so
    the same results bit for bit."""
    case = METRIC_COPY_CASES[name]
    print(f"[gpu] mixed without the metric copy {name}", flush=True)
    s = lesmi.Solver(case, prec=1)
    got = []
    for use in (True, False):
        assert lesmi.les_debug_metric_copy(s.ctx, use)
        Q = s.upload(case["Q"])
        step = s.rk_step(Q, 0.0, want_dt=True, want_norms=True)
        adv = s.advance(Q, 3, want_dt=True, want_norms=True)
        got.append((s.download(Q), step[0], step[1], adv[0], adv[1]))
    assert np.isfinite(I.interior(got[0][0])).all()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    s.close()


@pytest.mark.parametrize("shape", [(5, 5, 5), (23, 7, 6), (37, 15, 9)])
def test_residual_clears_shell(lesmi, shape):
    """les_residual writes every element of R: the residual at the interior
    nodes, and 0 in the ghosts, the row padding and the field's tail (rows of
    one and of several 16-element groups)."""
    import torch
    case = I.jet_case(*shape, seed=3)
    print(f"[gpu] residual shell {shape}", flush=True)
    s = lesmi.Solver(case)
    Q = s.upload(case["Q"])
    R = torch.full((5 * s.fe,), float("nan"), dtype=torch.float64, device="cuda")
    lesmi.les_residual(s.ctx, Q.data_ptr(), R.data_ptr())
    torch.cuda.synchronize()
    assert torch.isfinite(R).all()
    inner = s.download(R)[(slice(None), slice(2, -2), slice(2, -2), slice(2, -2))]
    assert np.count_nonzero(R.cpu().numpy()) == np.count_nonzero(inner) > 0
    s.close()


@pytest.mark.parametrize("shape,seg", [((61, 29, 23), "5"), ((31, 15, 9), "4"), ((93, 43, 17), ""),
                                       ((40, 20, 12), "7"), ((61, 29, 23), "40"), ((93, 43, 37), "200")])
def test_fused_matches_reference_kernel(lesmi, shape, seg, monkeypatch):
    """tiles 30 x 14 in (i, j): every shape leaves a ragged last tile; the
    segment sizes (tile-planes per persistent block) put segment starts and
    ends inside k and segments that span two tiles.  A share larger than nk
    (the last two cases) switches the blocks to round-robin (chunk, tile)
    segments, the schedule of the largest shards."""
    if seg:
        monkeypatch.setenv("LES_SEG", seg)
    else:
        monkeypatch.delenv("LES_SEG", raising=False)
    chunk = seg
    ni, nj, nk = shape
    case = I.jet_case(ni, nj, nk, seed=11)
    print(f"[gpu] fused vs reference {shape} chunk={chunk or 'auto'}", flush=True)
    a = lesmi.Solver(case)
    b = lesmi.Solver(case)
    b.use_reference(True)
    Qa = a.upload(case["Q"])
    Qb = b.upload(case["Q"])
    for _ in range(2):
        dta, na = a.rk_step(Qa, 0.0, want_dt=True, want_norms=True)
        dtb, nb = b.rk_step(Qb, 0.0, want_dt=True, want_norms=True)
        assert dta == dtb or abs(dta - dtb) <= 1e-15 * dtb
        assert np.allclose(na, nb, rtol=1e-11, atol=0)
    ga, gb = a.download(Qa), b.download(Qb)
    assert (_rel(ga, gb) <= 1e-13).all(), _rel(ga, gb)
    assert (_rel(ga - case["Q"], gb - case["Q"]) <= 1e-10).all()
    a.close()
    b.close()


def test_fused_matches_oracle_periodic_odd(orc, lesmi):
    n = (47, 33, 19)
    xyz = I.wavy_grid(*n, L=(2.0, 1.5, 1.0), amp=0.3)
    Q = I.smooth_state(*n, seed=21, amp=0.1)
    case = I.periodic_case(*n, xyz, Q, mu_ref=3e-3, sgs=1)
    s = lesmi.Solver(case)
    Qd = s.upload(Q)
    m = orc.metrics(case)
    Qo = Q
    for _ in range(3):
        s.rk_step(Qd)
        Qo, _, _, _ = orc.rk_step(case, m, Qo)
    assert (_rel(s.download(Qd), Qo) <= 1e-12).all()
    s.close()


# Mixed precision (FP32 stage states, fluxes and dissipation; FP64 Q^n,
# update, metrics and reductions).  Error of Q against the FP64 oracle per
# field, relative to the field's scale: max|rho| for rho, max|e| for e and
# the largest momentum component for the three momenta (a component that
# starts at zero, like rho w in the TGV, has no scale of its own).  Bound:
# FP32 rounding (6e-8) of the stage states and of flux terms up to ~1e3
# times the residual (Mach 0.1), accumulated over the steps: 2e-6.
MIXED_BOUND = 2e-6


@pytest.mark.parametrize("name,steps", [("tgv32", 10), ("jet150x40x20", 3)])
def test_mixed_precision_error(orc, lesmi, name, steps):
    case = I.tgv_case(32) if name == "tgv32" else I.jet_case(150, 40, 20, seed=4)
    s = lesmi.Solver(case, prec=lesmi.LES_MIXED)
    Q = s.upload(case["Q"])
    m = orc.metrics(case)
    Qo = case["Q"]
    for _ in range(steps):
        dt, norms = s.rk_step(Q, 0.0, want_dt=True, want_norms=True)
        Qo, dto, no, _ = orc.rk_step(case, m, Qo)
        assert abs(dt - dto) <= 1e-6 * dto  # dt from the FP64 state
    Qg = s.download(Q)
    d = I.interior(Qg) - I.interior(Qo)
    scale = np.abs(I.interior(Qo)).reshape(5, -1).max(1)
    scale[1:4] = scale[1:4].max()
    linf = np.abs(d).reshape(5, -1).max(1) / scale
    l2 = np.sqrt((d ** 2).reshape(5, -1).mean(1)) / scale
    print(f"[gpu] mixed {name}: Linf {linf} L2 {l2}", flush=True)
    assert (linf <= MIXED_BOUND).all(), linf
    assert np.isfinite(norms).all()
    s.close()


@pytest.mark.parametrize("shape", [(61, 29, 23), (31, 15, 9)])
def test_residual_fused_matches_reference(lesmi, shape):
    """les_residual through the fused kernel (the default) against the
    reference kernel, values and norms, with a source plane."""
    import torch
    ni, nj, nk = shape
    case = I.jet_case(ni, nj, nk, seed=13)
    print(f"[gpu] residual fused vs reference {shape}", flush=True)
    f = torch.from_numpy(1e-3 * np.random.default_rng(3).uniform(-1, 1, size=(5, nk, nj))).cuda()
    out = []
    for ref in (False, True):
        s = lesmi.Solver(case)
        s.use_reference(ref)
        s.set_forcing(f, ni // 3)
        R, norms = s.residual(s.upload(case["Q"]), want_norms=True)
        out.append((s.download(R), np.asarray(norms)))
        s.close()
    (ga, na), (gb, nb) = out
    assert (_rel(ga, gb) <= 1e-13).all(), _rel(ga, gb)
    assert np.allclose(na, nb, rtol=1e-11, atol=0)
