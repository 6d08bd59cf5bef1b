"""GPU parity of the solve-from-scratch step (lst_step_solve): U^{-T} is not
carried; each step forms A = U_new^T, factors it with partial pivoting and
solves A Z = H (section 3.5, last paragraph).  Same bars as the Woodbury step
against the explicit-W oracle, plus agreement with lst_step on the same inputs.
"""
import numpy as np
import pytest
import torch

from parity_util import rel, run_parity
from synth import Workload, WorkloadConfig

pytestmark = pytest.mark.gpu

TOL_STEP = 1e-4
TOL_W = 1e-3


def _cfg(**kw):
    base = dict(name="solve", D=5003, d=70, m=13, K=7, loss="squared", lr=1e-2, steps=30,
                idx_dist="uniform", distinct=False, val_dist="normal", entropy=401)
    base.update(kw)
    return WorkloadConfig(**base)


def _assert(reports, W_rel):
    worst = {k: max(getattr(r, k) for r in reports)
             for k in ("loss_rel", "loss_term_rel", "grad_rel", "grad_term_rel")}
    print(f"steps={len(reports)} " + " ".join(f"{k}={v:.2e}" for k, v in worst.items())
          + f" W rel={W_rel:.2e}", flush=True)
    for r in reports:
        assert r.loss_term_rel <= TOL_STEP, r
        assert r.grad_rel <= TOL_STEP, r
        assert r.grad_term_rel <= TOL_STEP, r
        assert r.rows_equal, r
    assert W_rel <= TOL_W, W_rel


@pytest.mark.parametrize("kw", [
    dict(d=70, m=13, K=7, pad_frac=0.2, dup_frac=0.3),        # rows not 16-byte aligned
    dict(d=37, m=1, K=5),                                      # one example, one ragged panel
    dict(d=130, m=150, K=30, idx_dist="zipf", zipf_s=1.1),     # m > 128, hot rows
    dict(d=96, m=20, K=1, loss="spherical", lr=1e-3, idx_dist="zipf", val_dist="one",
         distinct=True),
])
def test_step_solve_matches_oracle(gpu_lib, kw):
    cfg = _cfg(**kw, entropy=401 + kw["d"] + kw["m"])
    reports, W_rel, _ = run_parity(cfg, 30 if kw["m"] <= 20 else 10, solve=True,
                                   V_check_untouched=True)
    _assert(reports, W_rel)


def test_step_solve_paper_shape(gpu_lib):
    """D = 200000, d = 500, m = 128, K = 10 (the benchmarked shape), 20 steps."""
    cfg = _cfg(D=200000, d=500, m=128, K=10, lr=1e-3, distinct=True, entropy=411)
    reports, W_rel, _ = run_parity(cfg, 20, solve=True)
    _assert(reports, W_rel)


def test_step_solve_agrees_with_woodbury(gpu_lib):
    """The two forms of the step on the same inputs: the same loss, gradient and W
    to fp32 rounding."""
    import paper_1412_7091_amd as lst

    cfg = _cfg(D=4001, d=200, m=64, K=6, lr=5e-3, entropy=412)
    wl = Workload(cfg)
    dev = torch.device("cuda:0")
    V0 = torch.from_numpy(wl.init_V()).to(dev)
    a = lst.FactoredOutputLayer(V0, m_max=cfg.m, K_max=cfg.K)
    b = lst.FactoredOutputLayer(V0, m_max=cfg.m, K_max=cfg.K)
    for s in range(12):
        H, idx, val = (torch.from_numpy(x).to(dev) for x in wl.batch(s))
        la, ga = a.step(H, idx, val, cfg.lr)
        lb, gb = b.step_solve(H, idx, val, cfg.lr)
        assert a.sync() == 0 and b.sync() == 0
        assert rel(lb.cpu().numpy(), la.cpu().numpy()) < 1e-5
        assert rel(gb.cpu().numpy(), ga.cpu().numpy()) < 1e-5
    Wa = a.materialize_W().cpu().numpy()
    Wb = b.materialize_W().cpu().numpy()
    print(f"W rel {rel(Wb, Wa):.2e}", flush=True)
    assert rel(Wb, Wa) < 1e-5
    Qa, Ua, _ = a.get_state()
    Qb, Ub, _ = b.get_state()
    assert rel(Qb.cpu().numpy(), Qa.cpu().numpy()) < 1e-5
    assert rel(Ub.cpu().numpy(), Ua.cpu().numpy()) < 1e-5


def test_step_solve_leaves_uinvt_stale_until_restore(gpu_lib):
    import paper_1412_7091_amd as lst

    cfg = _cfg(D=1500, d=40, m=8, K=4, entropy=413)
    wl = Workload(cfg)
    dev = torch.device("cuda:0")
    layer = lst.FactoredOutputLayer(torch.from_numpy(wl.init_V()).to(dev), m_max=cfg.m,
                                    K_max=cfg.K)
    H, idx, val = (torch.from_numpy(x).to(dev) for x in wl.batch(0))
    layer.step_solve(H, idx, val, cfg.lr)
    assert layer.sync() == 0
    with pytest.raises(lst.LstError) as e:
        layer.step(H, idx, val, cfg.lr)
    assert e.value.code == lst.LST_ESTATE
    with pytest.raises(lst.LstError) as e:
        layer.stabilize()
    assert e.value.code == lst.LST_ESTATE
    W1 = layer.materialize_W().cpu().numpy()
    layer.restore()
    assert rel(layer.materialize_W().cpu().numpy(), W1) < 1e-5
    layer.step(H, idx, val, cfg.lr)
    assert layer.sync() == 0


def test_step_solve_singular(gpu_lib):
    """U = I, lr = 1/8, h = (2, 0, ...): U_new = I - 2 lr h h^T has a zero row and
    column, so the factorisation meets a zero pivot; nothing is updated."""
    import paper_1412_7091_amd as lst

    d, D = 8, 100
    dev = torch.device("cuda:0")
    V0 = torch.from_numpy(Workload(_cfg(D=D, d=d, m=1, K=1)).init_V()).to(dev)
    layer = lst.FactoredOutputLayer(V0, m_max=1, K_max=1)
    before = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    H = torch.zeros((1, d), dtype=torch.float32, device=dev)
    H[0, 0] = 2.0
    idx = torch.tensor([[3]], dtype=torch.int32, device=dev)
    val = torch.tensor([[1.0]], dtype=torch.float32, device=dev)
    layer.step_solve(H, idx, val, 0.125)
    assert layer.sync() == lst.LST_ESINGULAR
    after = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    for x, y in zip(before, after):
        assert torch.equal(x, y)


def test_step_solve_refuses_wide_state(gpu_lib):
    import paper_1412_7091_amd as lst

    dev = torch.device("cuda:0")
    V0 = torch.randn((50, 1100), device=dev) * 0.01
    layer = lst.FactoredOutputLayer(V0, m_max=2, K_max=1)
    H = torch.randn((2, 1100), device=dev)
    idx = torch.zeros((2, 1), dtype=torch.int32, device=dev)
    val = torch.ones((2, 1), device=dev)
    with pytest.raises(lst.LstError) as e:
        layer.step_solve(H, idx, val, 1e-3)
    assert e.value.code == lst.LST_EINVAL


@pytest.mark.parametrize("d,m", [(1, 1), (2, 3), (16, 5), (31, 17), (32, 16), (33, 1), (64, 33),
                                 (100, 40), (255, 15), (256, 130), (257, 31), (288, 16), (301, 77),
                                 (511, 2), (512, 128), (513, 48), (775, 20), (1023, 17),
                                 (1024, 100)])
def test_step_solve_row_solutions(gpu_lib, d, m):
    """Z = U_new^{-T} H itself, at the edges of panels (32), diagonal blocks (16), thread
    counts (256, 512, 1024) and example blocks (16), for an orthogonal U whose factorisation
    needs row interchanges at nearly every step.  With V = 0 and one target of its own per
    example, V_new holds 2 lr y z_i in the target's row.  Bound: the backward error of
    Gaussian elimination with partial pivoting, growth times d eps, with the d^(2/3) growth of
    random matrices, and cond(U_new) < 2."""
    import paper_1412_7091_amd as lst

    rng = np.random.default_rng(1000 * d + m)
    q, r = np.linalg.qr(rng.standard_normal((d, d)))
    U = np.ascontiguousarray(q * np.sign(np.diag(r)), dtype=np.float32)
    H = (rng.standard_normal((m, d)) / np.sqrt(d)).astype(np.float32)
    # 2 lr ||H^T H|| <= 1/2
    lr = np.float32(0.25 / max(1.0, np.linalg.norm(H.astype(np.float64), 2) ** 2))
    D = m + 3
    idx = rng.permutation(D)[:m].astype(np.int32).reshape(m, 1)
    val = (1.0 + rng.random((m, 1))).astype(np.float32)
    dev = torch.device("cuda:0")
    layer = lst.FactoredOutputLayer(torch.zeros((D, d), device=dev), torch.from_numpy(U).to(dev),
                                    m_max=m, K_max=1)
    layer.step_solve(*(torch.from_numpy(x).to(dev) for x in (H, idx, val)), float(lr))
    assert layer.sync() == 0
    V = layer.get_V().cpu().numpy().astype(np.float64)
    H64, U64 = H.astype(np.float64), U.astype(np.float64)
    U_new = U64 - 2.0 * float(lr) * (U64 @ H64.T) @ H64
    Z = np.linalg.solve(U_new.T, H64.T).T
    want = np.zeros((D, d))
    want[idx[:, 0]] = 2.0 * float(lr) * val.astype(np.float64) * Z
    err = np.linalg.norm(V - want) / np.linalg.norm(want)
    bound = 4.0 * d ** (2.0 / 3.0) * np.sqrt(d) * 2.0 ** -24 + 4.0 * 2.0 ** -24
    print(f"d={d} m={m}: {err:.2e} (bound {bound:.2e})", flush=True)
    assert err <= bound
    layer.close()


# columns in the first and last of the four waves' shares of a panel (8 columns each), past the
# first panel and at the end; d = 600 and 1024 start with panels of more than 512 rows
@pytest.mark.parametrize("d,col", [(8, 0), (8, 7), (100, 3), (100, 12), (100, 31), (100, 32),
                                   (100, 99), (300, 17), (300, 250), (600, 5), (600, 29),
                                   (600, 90), (600, 200), (600, 599), (1024, 0), (1024, 31),
                                   (1024, 500), (1024, 1023)])
@pytest.mark.parametrize("pivot", ["zero", "infinite"])
def test_step_solve_singular_columns(gpu_lib, d, col, pivot):
    """A pivot that vanishes, or is not finite, in column `col` of A = U_new^T only: U is a
    permutation and h lies along one unit vector, so U_new = U but for one entry, 1 - 8 lr
    (h = 2 e_j): 0 at lr = 1/8, minus infinity at lr = 3e38.  Nothing is updated."""
    import paper_1412_7091_amd as lst

    rng = np.random.default_rng(d + col)
    perm = rng.permutation(d)
    U = np.zeros((d, d), np.float32)
    U[np.arange(d), perm] = 1.0
    H = np.zeros((1, d), np.float32)
    H[0, perm[col]] = 2.0
    dev = torch.device("cuda:0")
    V0 = torch.from_numpy((rng.standard_normal((40, d)) / np.sqrt(d)).astype(np.float32)).to(dev)
    layer = lst.FactoredOutputLayer(V0, torch.from_numpy(U).to(dev), m_max=1, K_max=1)
    before = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    idx = torch.tensor([[3]], dtype=torch.int32, device=dev)
    val = torch.tensor([[1.0]], dtype=torch.float32, device=dev)
    layer.step_solve(torch.from_numpy(H).to(dev), idx, val, 0.125 if pivot == "zero" else 3e38)
    assert layer.sync() == lst.LST_ESINGULAR
    after = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    for x, y in zip(before, after):
        assert torch.equal(x, y)
    # and the next step of the same state is right
    lr = 0.0625
    layer.step_solve(torch.from_numpy(H).to(dev), idx, val, lr)
    assert layer.sync() == 0
    U_new = U.astype(np.float64)
    U_new[col, perm[col]] = 1.0 - 8.0 * lr
    assert rel(layer.get_state()[1].cpu().numpy(), U_new) < 1e-6
    layer.close()


@pytest.mark.parametrize("d", [100, 600])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_step_solve_nonfinite_example(gpu_lib, d, bad):
    """An example that is not finite: reported by its loss, the factorisation of a U_new full of
    NaN ends, and nothing is updated."""
    import paper_1412_7091_amd as lst

    cfg = _cfg(D=300, d=d, m=5, K=2, entropy=430 + d)
    wl = Workload(cfg)
    dev = torch.device("cuda:0")
    layer = lst.FactoredOutputLayer(torch.from_numpy(wl.init_V()).to(dev), m_max=5, K_max=2)
    before = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    H, idx, val = (torch.from_numpy(x).to(dev) for x in wl.batch(0))
    H[2, d // 2] = bad
    layer.step_solve(H, idx, val, cfg.lr)
    assert layer.sync() == lst.LST_ENONFINITE
    after = [x.clone() for x in layer.get_state()[:2]] + [layer.get_V().clone()]
    for x, y in zip(before, after):
        assert torch.equal(x, y)
    layer.close()
