"""GPU learned-closure kernels vs the oracle: residual generation (pairs,
features, normalised residuals), the BF16 matrix-core network's forward
pass and per-step gradients (against the FP64 oracle with the same bfloat16
rounding points), the Adam update, and that training on the method's own
residuals lowers the loss."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from oracle import mlp
import workloads
from paper_1211_2293_amd import treecode
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


def _ctx(w, lc=16):
    tc = treecode.Treecode(3, leaf_cap=lc)
    pos, mass = to_dev(w.pos), to_dev(w.mass)
    tc.build(pos, mass)
    tc.moments()
    return tc, (pos, mass)


@pytest.fixture(scope="module")
def plummer():
    w = workloads.plummer_sphere(20000, seed=90)
    tc, keep = _ctx(w)
    return w, tc, keep


def test_residuals_match_oracle(plummer):
    w, tc, _ = plummer
    targets = workloads.sample_indices(w.n, 64, seed=203)
    feat, y, cell = tc.residuals(0.9, 1e-2, to_dev(targets.astype(np.int32)))
    feat, y, cell = feat.cpu().numpy(), y.cpu().numpy(), cell.cpu().numpy()
    t = oracle.Tree(w.pos, w.mass, 16)
    r = t.residuals(0.9, 1e-2, targets)
    assert len(cell) == len(r["cell"]) and len(cell) > 64 * 50
    off = np.concatenate([[0], np.cumsum(r["count"])])
    for k in range(len(targets)):
        a, b = off[k], off[k + 1]
        og = np.argsort(cell[a:b])
        oo = np.argsort(r["cell"][a:b])
        np.testing.assert_array_equal(cell[a:b][og], r["cell"][a:b][oo])
        np.testing.assert_allclose(feat[a:b][og], r["feat"][a:b][oo], rtol=1e-6, atol=1e-6)
        ref = r["y"][a:b][oo]
        assert np.all(np.abs(y[a:b][og] - ref) <= 1e-6 * np.abs(ref) + 1e-9)


@pytest.mark.parametrize("n,nt,part,dtype", [(2, 2, 1.0, np.float32), (300, 300, 1.0, np.float32),
                                             (300, 1, 1.0, np.float64), (4000, 4000, 1.0, np.float32),
                                             (4000, 1500, 0.37, np.float64), (40000, 7, 1.0, np.float32),
                                             (40000, 9, 0.01, np.float32), (40000, 11, 1.0, np.float64)])
def test_residual_pairs_at_every_split(n, nt, part, dtype):
    """Cells of one body up to a quarter of the system, met by one to thousands
    of targets: runs of a cell of every length, and lists that fill the given
    arrays only in part.  The bounds are the ones of the oracle's test: FP64
    sums, rounded once."""
    w = workloads.plummer_sphere(n, seed=300 + n)
    tc = treecode.Treecode(3, leaf_cap=16)
    keep = to_dev(w.pos.astype(dtype)), to_dev(w.mass.astype(dtype))
    tc.build(*keep)
    tc.moments()
    targets = np.random.default_rng(n).permutation(n)[:nt].astype(np.int32)
    full = tc.residuals(0.9, 1e-2, to_dev(targets))
    cap = int(np.ceil(part * len(full[2])))
    feat, y, cell = tc.residuals(0.9, 1e-2, to_dev(targets), cap=cap) if part < 1.0 else full
    feat, y, cell = feat.cpu().numpy(), y.cpu().numpy(), cell.cpu().numpy()
    # arrays with room for more: what lies past the pairs is left alone
    spare = [torch.full((len(full[2]) + 5, *t.shape[1:]), 7, dtype=t.dtype, device="cuda") for t in full]
    n_out = C.c_int64()
    assert treecode.lib().tc_residuals(tc._h, 0.9, 1e-2, to_dev(targets).data_ptr(), nt, *(t.data_ptr() for t in spare),
                                       len(spare[2]), C.byref(n_out)) == 0
    torch.cuda.synchronize()
    for t, u in zip(spare, full):
        assert torch.equal(t[:len(u)], u) and bool((t[len(u):] == 7).all())
    r = oracle.Tree(w.pos, w.mass, 16).residuals(0.9, 1e-2, targets)
    off = np.concatenate([[0], np.cumsum(r["count"])])
    assert len(full[2]) == off[-1]
    np.testing.assert_array_equal(cell[:cap], full[2].cpu().numpy()[:cap])
    for k in range(nt):
        a, b = off[k], off[k + 1]
        if b > cap:
            break
        og, oo = np.argsort(cell[a:b]), np.argsort(r["cell"][a:b])
        np.testing.assert_array_equal(cell[a:b][og], r["cell"][a:b][oo])
        np.testing.assert_allclose(feat[a:b][og], r["feat"][a:b][oo], rtol=1e-6, atol=1e-6)
        ref = r["y"][a:b][oo]
        assert np.all(np.abs(y[a:b][og] - ref) <= 1e-6 * np.abs(ref) + 1e-9)


def _features(n=3000, seed=91):
    rng = np.random.default_rng(seed)
    f = np.concatenate([rng.normal(size=(n, 9)) * [1, 1, 1, .3, .3, .3, .3, .3, .3],
                        rng.uniform(0, 8, (n, 1))], axis=1).astype(np.float32)
    y = (rng.normal(size=(n, 3)) * 0.02).astype(np.float32)
    return f, y


def test_forward_matches_bf16_oracle(plummer):
    _, tc, _ = plummer
    theta = mlp.init_params(seed=5)
    tc.mlp_load(to_dev(theta))
    f, _ = _features()
    out = tc.mlp_forward(to_dev(f)).cpu().numpy()
    ref, _ = mlp.forward(theta, f, bf16_ops=True)
    print(f"forward rel L2 {oracle.rel_l2(out, ref):.2e}", flush=True)
    assert oracle.rel_l2(out, ref) < 1e-3
    np.testing.assert_array_equal(tc.mlp_get().cpu().numpy(), theta)


def test_gradient_matches_bf16_oracle(plummer):
    _, tc, _ = plummer
    theta = mlp.init_params(seed=6)
    tc.mlp_load(to_dev(theta))
    f, y = _features(4000, seed=92)
    idx = np.random.default_rng(93).permutation(4000)[:2500].astype(np.int32)
    grad = torch.empty(mlp.NPARAM, dtype=torch.float32, device="cuda")
    loss = tc.mlp_step(to_dev(f), to_dev(y), to_dev(idx), lr=0.0, grad=grad)
    rl, rg = mlp.loss_and_grad(theta, f[idx], y[idx], bf16_ops=True)
    g = grad.cpu().numpy()
    print(f"loss {loss:.6e} vs {rl:.6e}; grad rel L2 {oracle.rel_l2(g, rg):.2e}", flush=True)
    assert abs(loss - rl) <= 1e-4 * rl
    assert oracle.rel_l2(g, rg) < 1e-3
    # lr = 0 leaves the parameters unchanged
    np.testing.assert_array_equal(tc.mlp_get().cpu().numpy(), theta)


@pytest.mark.parametrize("nb", [1, 15, 16, 17, 63, 64, 65, 129, 1000, 1025])
def test_gradient_at_batch_edges(plummer, nb):
    """Batches that fill a wave's 16 samples, a block's 64 and the sixteen
    blocks' partials summed at a time, and one sample either side, with rows
    outside the features dropped (their index flagged): the same bar as above."""
    _, tc, keep = plummer
    theta = mlp.init_params(seed=8)
    tc.mlp_load(to_dev(theta))
    f, y = _features(1100, seed=96)
    rng = np.random.default_rng(97)
    idx = rng.integers(0, len(f), nb).astype(np.int32)
    grad = torch.empty(mlp.NPARAM, dtype=torch.float32, device="cuda")
    loss = tc.mlp_step(to_dev(f), to_dev(y), to_dev(idx), lr=0.0, grad=grad)
    rl, rg = mlp.loss_and_grad(theta, f[idx], y[idx], bf16_ops=True)
    assert abs(loss - rl) <= 1e-4 * rl
    assert oracle.rel_l2(grad.cpu().numpy(), rg) < 1e-3
    if nb == 129:
        # a dropped sample adds nothing: the sums are over the others, the mean over all
        bad = idx.copy()
        bad[[0, 77]] = (-1, len(f))
        tc.mlp_step(to_dev(f), to_dev(y), to_dev(bad), lr=0.0, grad=grad)
        ok = np.delete(idx, [0, 77])
        _, rg = mlp.loss_and_grad(theta, f[ok], y[ok], bf16_ops=True)
        assert oracle.rel_l2(grad.cpu().numpy(), rg * (len(ok) / nb)) < 1e-2
        assert tc.status() == treecode.TC_EINVAL
        tc.build(*keep)                       # clears the flag
        tc.moments()
        tc.mlp_load(to_dev(theta))


def test_adam_step_matches_oracle(plummer):
    _, tc, _ = plummer
    theta = mlp.init_params(seed=7)
    tc.mlp_load(to_dev(theta))
    f, y = _features(1000, seed=94)
    grad = torch.empty(mlp.NPARAM, dtype=torch.float32, device="cuda")
    tc.mlp_step(to_dev(f), to_dev(y), lr=1e-3, grad=grad)
    g = grad.cpu().numpy().astype(np.float64)
    ref, _, _ = mlp.adam(theta.astype(np.float64), g, np.zeros(mlp.NPARAM), np.zeros(mlp.NPARAM), 1, lr=1e-3)
    np.testing.assert_allclose(tc.mlp_get().cpu().numpy(), ref, rtol=0, atol=2e-6)


def test_training_on_residuals_lowers_the_loss_and_the_force_error():
    """Train on the method's own residuals (a 65,536-body Plummer sphere,
    pairs at theta = 0.9), then show what the network gains at force level:
    the learned walk at theta_L = 0.8 (every learned cell kept) has a
    relative force error against the FP64 direct sum well below the plain
    walk's at the same theta_L."""
    from paper_1211_2293_amd import closure
    w = workloads.plummer_sphere(65536, seed=95)
    tc, keep = _ctx(w)
    f_tr, y_tr = closure.residual_pairs(tc, 0.9, 1e-2, workloads.sample_indices(w.n, 512, seed=203))
    f_va, y_va = closure.residual_pairs(tc, 0.9, 1e-2, workloads.sample_indices(w.n, 128, seed=204))
    p0, order = workloads.training_draws(f_tr.shape[0], 200, 4096)
    st = closure.train(tc, f_tr, y_tr, p0, order, epochs=200, lr=1e-2, lr_final=1e-5, val=(f_va, y_va))
    quad = float(((closure.quadrupole_prediction(f_va) - y_va) ** 2).mean())
    print(f"pairs {st['pairs']}, {st['steps']} steps; loss {st['loss_first']:.3e} -> {st['loss_last']:.3e}; "
          f"validation {st['val_mse']:.3e} vs zero predictor {st['val_mse_zero']:.3e}, "
          f"analytic quadrupole {quad:.3e}", flush=True)
    assert st["loss_last"] < 0.5 * st["loss_first"]
    assert st["val_mse"] < 0.2 * st["val_mse_zero"]
    sample = workloads.sample_indices(w.n, 2048, seed=104)
    ref, _ = tc.direct(to_dev(sample.astype(np.int32)), G=1.0, eps=1e-2)
    ref = ref.cpu().numpy()
    tc.walk(0.8)
    plain, _ = tc.forces(1.0, 1e-2)
    learned, _ = tc.forces_learned(0.8, 0.5, float("inf"), eps=1e-2)
    tc.walk(0.5)
    plain_p, _ = tc.forces(1.0, 1e-2)
    e_plain = oracle.rel_l2(plain.cpu().numpy()[sample], ref)
    e_learn = oracle.rel_l2(learned.cpu().numpy()[sample], ref)
    e_p = oracle.rel_l2(plain_p.cpu().numpy()[sample], ref)
    print(f"E vs direct: plain theta 0.8 {e_plain:.3e}, learned 0.8/0.5 {e_learn:.3e}, plain 0.5 {e_p:.3e}",
          flush=True)
    assert e_learn < 0.8 * e_plain


@pytest.fixture(scope="module")
def learned_case():
    """A 4000-body Plummer sphere, a random network scaled so corrections
    stay a few percent of the force, and the oracle's learned walk."""
    w = workloads.plummer_sphere(4000, seed=97)
    tc, keep = _ctx(w)
    p = mlp.unflatten(mlp.init_params(seed=9).astype(np.float64))
    p["W3"] *= 0.2
    theta = mlp.flatten(p).astype(np.float32)
    tc.mlp_load(to_dev(theta))
    t = oracle.Tree(w.pos, w.mass, 16)
    ref = mlp.learned_corrections(t, 0.9, 0.5, theta, G=1.0)
    return w, tc, keep, t, theta, ref


def test_learned_walk_tau_zero_is_plain_walk_at_theta_p(learned_case):
    w, tc, _, t, _, ref = learned_case
    acc, pot = tc.forces_learned(0.9, 0.5, 0.0, eps=1e-2)
    m2p, p2p = (v.cpu().numpy() for v in tc.counts())
    kept, fell = (v.cpu().numpy() for v in tc.learned_counts())
    gb, gc = t.groups(64, 1024)
    rm2p, rp2p = t.walk_counts_groups(0.5, gb, gc)
    np.testing.assert_array_equal(m2p, rm2p)
    np.testing.assert_array_equal(p2p, rp2p)
    assert np.all(kept == 0)
    np.testing.assert_array_equal(fell, ref["per_group"])
    a, ph = t.forces_groups(0.5, gb, gc, eps=1e-2)
    ea, ep = oracle.rel_l2(acc.cpu().numpy(), a), oracle.rel_l2(pot.cpu().numpy(), ph)
    print(f"tau=0: acc {ea:.2e} pot {ep:.2e}; learned cells {ref['per_group'].sum()}", flush=True)
    assert ea < 1e-5 and ep < 1e-5


def test_learned_walk_tau_inf_is_theta_l_plus_corrections(learned_case):
    w, tc, _, t, _, ref = learned_case
    acc, pot = tc.forces_learned(0.9, 0.5, float("inf"), eps=1e-2)
    m2p, p2p = (v.cpu().numpy() for v in tc.counts())
    kept, fell = (v.cpu().numpy() for v in tc.learned_counts())
    gb, gc = t.groups(64, 1024)
    rm2p, rp2p = t.walk_counts_groups(0.9, gb, gc)
    np.testing.assert_array_equal(m2p, rm2p)
    np.testing.assert_array_equal(p2p, rp2p)
    np.testing.assert_array_equal(kept, ref["per_group"])
    assert np.all(fell == 0)
    a, ph = t.forces_groups(0.9, gb, gc, eps=1e-2)
    g_acc = acc.cpu().numpy()
    total = oracle.rel_l2(g_acc, a + ref["corr"])
    corr = oracle.rel_l2(g_acc - a, ref["corr"])
    ep = oracle.rel_l2(pot.cpu().numpy(), ph)
    size = np.linalg.norm(ref["corr"]) / np.linalg.norm(a)
    print(f"tau=inf: total {total:.2e}, corrections {corr:.2e} (|corr|/|acc| {size:.2e}), pot {ep:.2e}", flush=True)
    assert size > 1e-3
    assert corr < 1e-2 and total < 1e-5 + 1e-2 * size and ep < 1e-5


def _median_tau_case(w, tc, t, theta, theta_l=0.9, theta_p=0.5, min_size=1e-3):
    """The GPU's learned walk at the median of the oracle's fallback
    statistics against the oracle's learned walk with the same tau: kept and
    fallen-back counts per group, and forces element by element, on every
    group whose learned cells all lie clear of tau (the statistic comes out
    of a BF16 network, FP32 on the GPU and FP64 in the oracle, so cells
    within 2% of tau may decide either way)."""
    ri = mlp.learned_walk(t, theta_l, theta_p, np.inf, theta, eps=w.eps)
    gm, pg = ri["pair_gmax"], ri["pair_group"]
    tau = float(np.median(gm))
    ref = mlp.learned_walk(t, theta_l, theta_p, tau, theta, eps=w.eps)
    acc, pot = tc.forces_learned(theta_l, theta_p, tau, eps=w.eps)
    kept, fell = (v.cpu().numpy() for v in tc.learned_counts())
    np.testing.assert_array_equal(kept + fell, ref["kept"] + ref["fell"])
    near = np.zeros(len(kept), bool)
    near[pg[np.abs(gm - tau) <= 0.02 * tau]] = True
    safe = ~near
    np.testing.assert_array_equal(kept[safe], ref["kept"][safe])
    np.testing.assert_array_equal(fell[safe], ref["fell"][safe])
    assert kept[safe].sum() > 0 and fell[safe].sum() > 0
    gb, gc = t.groups(64, 1024)
    perm = t.bodies()["perm"]
    sel = np.concatenate([perm[b:b + k] for b, k, ok in zip(gb, gc, safe) if ok])
    g_acc, g_pot = acc.cpu().numpy()[sel], pot.cpu().numpy()[sel]
    a, ph = ref["acc"][sel], ref["pot"][sel]
    a_plain, _ = t.forces_groups(theta_l, gb, gc, eps=w.eps)
    size = np.linalg.norm(ri["acc"][sel] - a_plain[sel]) / np.linalg.norm(a)
    ea, ep = oracle.rel_l2(g_acc, a), oracle.rel_l2(g_pot, ph)
    print(f"tau={tau:.3e}: kept {kept.sum()} fell {fell.sum()}; {safe.sum()}/{len(safe)} groups compared; "
          f"acc {ea:.2e} (|corr|/|acc| {size:.2e}), pot {ep:.2e}", flush=True)
    assert size > min_size
    assert ea < 1e-5 + 1e-2 * size and ep < 1e-5


def test_learned_walk_median_tau_plummer(learned_case):
    w, tc, _, t, theta, _ = learned_case
    _median_tau_case(w, tc, t, theta)


def test_learned_walk_median_tau_clustered_pareto_masses():
    """32 clumps with Pareto(2.35) masses: ln(M / mbar) of the learned cells
    spreads far wider than in an equal-mass sphere."""
    w = workloads.clustered(20000, seed=98)
    tc, keep = _ctx(w)
    theta = mlp.init_params(seed=12).astype(np.float32)
    tc.mlp_load(to_dev(theta))
    t = oracle.Tree(w.pos, w.mass, 16)
    # eps = 1e-3 and compact clumps: the learned cells' share of the force is
    # smaller than in the sphere, the bar 1e-5 + 1e-2 |corr| tighter
    _median_tau_case(w, tc, t, theta, theta_l=0.8, min_size=3e-4)


def test_plain_walk_theta_survives_a_learned_call(learned_case):
    """A learned evaluation computes its own opening radii; a later plain
    tc_forces walks at the theta of the last tc_walk again, bit for bit."""
    w, tc, _, _, _, _ = learned_case
    tc.walk(0.6)
    a1, p1 = tc.forces(1.0, 1e-2)
    a1, p1 = a1.cpu().numpy(), p1.cpu().numpy()
    tc.forces_learned(0.9, 0.5, float("inf"), eps=1e-2)
    a2, p2 = tc.forces(1.0, 1e-2)
    np.testing.assert_array_equal(a2.cpu().numpy(), a1)
    np.testing.assert_array_equal(p2.cpu().numpy(), p1)


def test_learned_leapfrog_step_matches_oracle():
    """One kick-drift-kick step with the learned walk (tc_set_closure) on
    FP64 state against oracle.kdk driven by the oracle's learned walk, then
    a plain step after switching the closure off."""
    w = workloads.plummer_sphere(4000, seed=99)
    x0, v0, m = (a.astype(np.float64) for a in (w.pos, w.vel, w.mass))
    pos, vel, mass = to_dev(x0), to_dev(v0), to_dev(m)
    tc = treecode.Treecode(3, leaf_cap=16)
    tc.build(pos, mass)
    tc.moments()
    p = mlp.unflatten(mlp.init_params(seed=13).astype(np.float64))
    p["W3"] *= 0.2
    theta = mlp.flatten(p).astype(np.float32)
    tc.mlp_load(to_dev(theta))
    tl, tp, eps, dt = 0.9, 0.5, 1e-2, 1e-3
    tc.set_closure(tl, tp, float("inf"))
    with pytest.raises(treecode.TcError):          # no force evaluation yet
        tc.leapfrog(dt, pos, vel)
    tc.forces_learned(tl, tp, float("inf"), eps=eps)
    tc.leapfrog(dt, pos, vel)
    acc1, _ = tc.forces_learned(tl, tp, float("inf"), eps=eps)
    kept, fell = (v.cpu().numpy() for v in tc.learned_counts())
    assert tc.status() == treecode.TC_OK

    def f(x):
        return mlp.learned_walk(oracle.Tree(x, m, 16), tl, tp, np.inf, theta, eps=eps)["acc"]

    a0 = f(x0)
    x1, v1, a1 = oracle.kdk(x0, v0, a0, dt, f)
    gx, gv = pos.cpu().numpy(), vel.cpu().numpy()
    ex, ev, ea = oracle.rel_l2(gx, x1), oracle.rel_l2(gv, v1), oracle.rel_l2(acc1.cpu().numpy(), a1)
    print(f"learned step: x {ex:.2e}, v {ev:.2e}, a(x') {ea:.2e}; kept {kept.sum()} fell {fell.sum()}", flush=True)
    t1 = oracle.Tree(x1, m, 16)
    plain_l, _ = t1.walk_forces(tl, eps=eps)
    size = oracle.rel_l2(a1, plain_l)                # corrections relative to the force
    assert kept.sum() > 0 and fell.sum() == 0 and size > 1e-3
    assert ex < 1e-10 and ev < 1e-6 and ea < 1e-5 + 1e-2 * size
    # switched off: the next step is the plain walk at the last tc_walk's theta
    tc.set_closure(None)
    with pytest.raises(treecode.TcError):          # no tc_walk has fixed a plain theta
        tc.leapfrog(dt, pos, vel)
    tc.walk(0.5)
    tc.forces(1.0, eps)
    tc.leapfrog(dt, pos, vel)
    a_pl, _ = tc.forces(1.0, eps)
    t2 = oracle.Tree(pos.cpu().numpy(), m, 16)
    ref, _ = t2.walk_forces(0.5, eps=eps)
    assert oracle.rel_l2(a_pl.cpu().numpy(), ref) < 1e-5


@pytest.mark.parametrize("n,theta_l,theta_p", [(70, 0.9, 0.3), (777, 1.0, 0.4), (9000, 0.3, 0.02)])
def test_learned_walk_by_blocks(n, theta_l, theta_p):
    """One or two groups of one to four tiles, and groups with more learned
    cells than the block's queue holds (512), kept and fallen back; the bounds
    are those of the walks above."""
    w = workloads.plummer_sphere(n, seed=500 + n)
    tc, keep = _ctx(w)
    p = mlp.unflatten(mlp.init_params(seed=9).astype(np.float64))
    p["W3"] *= 0.2
    theta = mlp.flatten(p).astype(np.float32)
    tc.mlp_load(to_dev(theta))
    t = oracle.Tree(w.pos, w.mass, 16)
    # (the oracle's network over the largest case's million pairs takes minutes:
    # its corrections are left out there)
    ref = mlp.learned_corrections(t, theta_l, theta_p, theta, G=1.0) if n < 9000 else None
    gb, gc = t.groups(64, 1024)
    learned = []
    for tau, th in ((0.0, theta_p), (float("inf"), theta_l)):
        acc, pot = tc.forces_learned(theta_l, theta_p, tau, eps=1e-2)
        m2p, p2p = (v.cpu().numpy() for v in tc.counts())
        kept, fell = (v.cpu().numpy() for v in tc.learned_counts())
        rm2p, rp2p = t.walk_counts_groups(th, gb, gc)
        np.testing.assert_array_equal(m2p, rm2p)
        np.testing.assert_array_equal(p2p, rp2p)
        assert np.all((kept if tau == 0.0 else fell) == 0)
        learned.append(fell if tau == 0.0 else kept)
        a, ph = t.forces_groups(th, gb, gc, eps=1e-2)
        ep = oracle.rel_l2(pot.cpu().numpy(), ph)
        assert ep < 1e-5
        if tau == 0.0 or ref is not None:
            size = 0.0 if tau == 0.0 else np.linalg.norm(ref["corr"]) / np.linalg.norm(a)
            ea = oracle.rel_l2(acc.cpu().numpy(), a if tau == 0.0 else a + ref["corr"])
            print(f"n={n} tau={tau}: acc {ea:.2e} pot {ep:.2e}, learned up to {learned[-1].max()}", flush=True)
            assert ea < 1e-5 + 1e-2 * size
    np.testing.assert_array_equal(learned[0], learned[1])
    if ref is not None:
        np.testing.assert_array_equal(learned[0], ref["per_group"])
    else:
        assert learned[0].max() > 512


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_residuals_under_a_softening_whose_square_overflows(dtype):
    """eps is finite, eps^2 is not: the exact sum and the monopole vanish, as
    1 / sqrt(inf) does, in cells summed by lanes, by a wave and by a block."""
    w = workloads.plummer_sphere(40000, seed=98)
    tc = treecode.Treecode(3, leaf_cap=16)
    keep = to_dev(w.pos.astype(dtype)), to_dev(w.mass.astype(dtype))
    tc.build(*keep)
    tc.moments()
    far = np.argsort(-np.linalg.norm(w.pos, axis=1))[:40].astype(np.int32)
    feat, y, cell = tc.residuals(1.0, 1e160, to_dev(far))
    count = tc.cells()["count"][cell.long()]
    assert int(count.max()) > 4096 and int(count.min()) < 128
    assert bool((y == 0.0).all()) and bool(torch.isfinite(feat).all())


@pytest.mark.parametrize("nt,dtype", [(600, np.float32), (7, np.float64)])
def test_residual_pairs_of_cells_that_share_keys(nt, dtype):
    """Cells past the first 16,128 in level order share 256 keys by target:
    accepted cells on both sides of that line, more targets than keys and
    fewer; the bounds are the ones of the oracle's test."""
    n = 120000
    w = workloads.plummer_sphere(n, seed=99)
    tc = treecode.Treecode(3, leaf_cap=4)
    keep = to_dev(w.pos.astype(dtype)), to_dev(w.mass.astype(dtype))
    tc.build(*keep)
    tc.moments()
    targets = np.random.default_rng(100).permutation(n)[:nt].astype(np.int32)
    feat, y, cell = (v.cpu().numpy() for v in tc.residuals(0.9, 1e-2, to_dev(targets)))
    t = oracle.Tree(w.pos, w.mass, 4)
    # level-order places: by level, pre-order within a level
    level = tc.cells(moments=False)["level"].cpu().numpy()
    place = np.empty(len(level), np.int64)
    place[np.argsort(level, kind="stable")] = np.arange(len(level))
    past = place[cell] >= 16128
    assert past.sum() > 3 * nt and (~past).sum() > 3 * nt
    r = t.residuals(0.9, 1e-2, targets)
    off = np.concatenate([[0], np.cumsum(r["count"])])
    assert len(cell) == off[-1]
    for k in range(nt):
        a, b = off[k], off[k + 1]
        og, oo = np.argsort(cell[a:b]), np.argsort(r["cell"][a:b])
        np.testing.assert_array_equal(cell[a:b][og], r["cell"][a:b][oo])
        np.testing.assert_allclose(feat[a:b][og], r["feat"][a:b][oo], rtol=1e-6, atol=1e-6)
        ref = r["y"][a:b][oo]
        assert np.all(np.abs(y[a:b][og] - ref) <= 1e-6 * np.abs(ref) + 1e-9)


@pytest.mark.parametrize("n", [1, 2, 40, 1023, 1024, 1025])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_residual_pairs_of_the_smallest_systems(n, dtype):
    """Both sides of the size up to which the pairs take one launch: pairs,
    features and residuals against the oracle, arrays that hold a part of the
    pairs, what lies past them, and targets outside the bodies."""
    w = workloads.plummer_sphere(n, seed=101)
    tc = treecode.Treecode(3, leaf_cap=2)
    keep = to_dev(w.pos.astype(dtype)), to_dev(w.mass.astype(dtype))
    tc.build(*keep)
    tc.moments()
    targets = np.random.default_rng(102).integers(0, n, min(n, 70)).astype(np.int32)
    full = tc.residuals(0.8, 1e-2, to_dev(targets))
    r = oracle.Tree(w.pos, w.mass, 2).residuals(0.8, 1e-2, targets)
    off = np.concatenate([[0], np.cumsum(r["count"])])
    assert len(full[2]) == off[-1]
    feat, y, cell = (v.cpu().numpy() for v in full)
    for k in range(len(targets)):
        a, b = off[k], off[k + 1]
        og, oo = np.argsort(cell[a:b]), np.argsort(r["cell"][a:b])
        np.testing.assert_array_equal(cell[a:b][og], r["cell"][a:b][oo])
        np.testing.assert_allclose(feat[a:b][og], r["feat"][a:b][oo], rtol=1e-6, atol=1e-6)
        ref = r["y"][a:b][oo]
        assert np.all(np.abs(y[a:b][og] - ref) <= 1e-6 * np.abs(ref) + 1e-9)
    if off[-1] < 2:
        return
    cap = int(off[-1]) // 2 + 1
    spare = [torch.full((cap + 7, *t.shape[1:]), 7, dtype=t.dtype, device="cuda") for t in full]
    n_out = C.c_int64()
    assert treecode.lib().tc_residuals(tc._h, 0.8, 1e-2, to_dev(targets).data_ptr(), len(targets),
                                       *(t.data_ptr() for t in spare), cap, C.byref(n_out)) == 0
    torch.cuda.synchronize()
    assert n_out.value == off[-1]
    for t, u in zip(spare, full):
        assert torch.equal(t[:cap], u[:cap]) and bool((t[cap:] == 7).all())
    bad = targets.copy()
    bad[[0, -1]] = (-1, n)
    got = tc.residuals(0.8, 1e-2, to_dev(bad))
    assert tc.status() == treecode.TC_EINVAL
    mid = slice(int(off[1]), int(off[-2]))
    for t, u in zip(got, full):
        assert torch.equal(t, u[mid])
