"""Chunk products with split operands, the carries and walks beside them, and the read-out: results against
the float64 oracle's at the edges of the tiles, for operands of very different size, and where a chunk
keeps its stored product."""
import os

import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2605_12683_amd as D  # noqa: E402
from gpu_util import oracle_model, rel_inf, say  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-4   # the project's normwise tolerance


@pytest.fixture(autouse=True)
def _chunk():
    os.environ.pop("DEER_CHUNK", None)
    yield
    os.environ.pop("DEER_CHUNK", None)


def _case(M, N, B, T, seed, a_range=(0.3, 0.75), w_norm=0.2):
    return W.random_plrnn_case(M, N, B, T, 0.2, seed, w_norm=w_norm, a_range=a_range)


# M: first and last width of each padded size, a width that is no multiple of 4 and one that is;
# chunks: shorter than the 8-step tile of the local kernel, one tile, one over the 64-step mask tile
@pytest.mark.parametrize("M,N,B,T,chunk,T_w", [
    (17, 3, 2, 40, 5, 0), (20, 20, 1, 130, 65, 0), (32, 8, 17, 64, 16, 9), (33, 33, 2, 200, 66, 0),
    (48, 12, 3, 65, 8, 64), (63, 5, 1, 257, 128, 3), (64, 64, 2, 1, 16, 0), (64, 0, 2, 90, 31, 0), (64, 64, 2, 300, 100, 120)])
def test_iterates(M, N, B, T, chunk, T_w):
    os.environ["DEER_CHUNK"] = str(chunk)
    c = _case(M, N or 3, B, T, 6000 + M + T)
    init = "teacher" if N else "zero"   # nothing observed: x is not read
    say("split iterates", M, N, B, T, chunk, T_w)
    rng = np.random.default_rng(M)
    z0 = rng.standard_normal((B, M)).astype(np.float32)
    for k in (1, 3):
        res = D.deer_solve(oracle_model(c), c.x, 0.2, N, fixed_iters=k, z0=z0, T_w=T_w, init=init)
        ref = O.newton(oracle_model(c), c.x, 0.2, N, fixed_iters=k, z0=z0, T_w=T_w, init=init)
        assert rel_inf(res["z"].cpu().numpy(), ref["z"]) < TOL


# weights far from one, a diagonal far below W, rows of very different size (units of the latents:
# test_gpu_units.py)
@pytest.mark.parametrize("M", [24, 64])
@pytest.mark.parametrize("kind", ["large", "huge", "tiny", "rows", "zero"])
def test_scales(M, kind):
    os.environ["DEER_CHUNK"] = "2" if kind == "huge" else "24"
    T = {"large": 60, "huge": 5}.get(kind, 96)
    c = _case(M, M, 2, T, 6100 + M)
    p = {k: v.copy() for k, v in c.params.items()}
    if kind == "large":        # products grow to ~1e30 within the sequence
        p["W"] *= 16.0
    elif kind == "huge":       # one step grows by ~2^20
        p["W"] *= np.float32(2.0 ** 21)
    elif kind == "tiny":       # products fall by ~2^-10 a step
        p["W"] *= 1e-3
        p["A"] *= 1e-3
    elif kind == "rows":
        p["W"] *= (2.0 ** -np.linspace(0, 18, M)).astype(np.float32)[:, None]
    else:
        p["W"] *= 0.0
        p["A"] *= 0.0
    m = {"kind": "plrnn", **p}
    x = c.x[:, :T + 1]
    say("split scales", M, kind)
    res = D.deer_solve(m, x, 0.2, M, fixed_iters=1, init="zero")
    ref = O.newton(m, x, 0.2, M, fixed_iters=1, init="zero")
    assert rel_inf(res["z"].cpu().numpy(), ref["z"]) < TOL


@pytest.mark.parametrize("M,bound", [(20, 0.0), (64, 0.0), (64, 0.05), (33, 0.05)])
def test_kept_products(M, bound):
    """Updates past convergence keep every chunk's product (no mask changes), and with a small step
    bound rejected updates re-form them with another damping at unchanged masks: the fixed point
    and a second, tighter solve from it agree with the rollout (a product kept wrongly would slow the
    solve, not move its result: the next two tests look at the iterates on the way)."""
    os.environ["DEER_CHUNK"] = "32"
    c = _case(M, M, 3, 500, 6200 + M, w_norm=0.35)
    m = oracle_model(c)
    ref = O.rollout(m, c.x, 0.2, M)
    say("split kept products", M, bound)
    res = D.deer_solve(m, c.x, 0.2, M, tol=1e-5, max_iter=5000, step_bound=bound)
    assert res["status"] == 0 and rel_inf(res["z"].cpu().numpy(), ref) < TOL
    more = D.deer_solve(m, c.x, 0.2, M, fixed_iters=8)
    assert rel_inf(more["z"].cpu().numpy(), ref) < 1e-5


def _chunked_newton(m, x, alpha, N, z, C, updates=0, passes=0, bound=0.0, stale=None):
    """Newton passes of one sequence in float64, the linear solve in chunks of C steps as the library does
    it: chunk products, carries, each chunk re-run from its carry with the pass's own Jacobians.  `updates`
    plain updates, or `passes` passes of the safeguarded loop (an update over bound (1 + max |z|) is
    rejected and tried again with damping 1 - om).  stale: products that should not be kept are, "masks"
    those of the first pass, "damping" those whose masks stand though the damping changed.  Returns z, the
    accepted updates and the smallest relative distance of an update from the bound."""
    T, M = z.shape[1:]
    z = z.astype(np.float64)
    p = 1.0 - O.forcing_weights(M, N, alpha)
    om, accepted, gap, P, old = 0.0, 0, np.inf, {}, None
    for _ in range(updates or passes):
        r, _, mask, _ = O.residual_and_masks(m, x, z, alpha, N)
        J = (1.0 - om) * O.jacobian_dense({k: np.asarray(v, np.float64) if k != "kind" else v for k, v in m.items()}, mask)[0] * p
        delta, cur = np.empty((T, M)), np.zeros(M)
        for t0 in range(0, T, C):
            t1 = min(t0 + C, T)
            keep = old is not None and (stale == "masks" or stale == "damping"
                                        and np.array_equal(old[0, t0:t1], mask[0, t0:t1]))
            if not keep:
                P[t0] = np.eye(M)
                for t in range(t0, t1):
                    P[t0] = J[t] @ P[t0]
            d, v = cur, np.zeros(M)
            for t in range(t0, t1):
                d, v = J[t] @ d - r[0, t], J[t] @ v - r[0, t]
                delta[t] = d
            cur = P[t0] @ cur + v
        old = mask
        e, lim = np.abs(delta).max(), bound * (1.0 + np.abs(z).max())
        if updates or om >= 1.0 or e <= lim:
            z[0] += delta
            accepted += 1
            om = 0.0 if om / 4 < 1e-4 else om / 4
        else:
            om = 1.0 / 64 if om == 0.0 else min(1.0, om * 4)
        if passes:
            gap = min(gap, abs(e / lim - 1.0))
    return z, accepted, gap


def _stale_case(kind, M, L, w_norm):
    """A wide-awake model and a start far from the solution: masks change in every pass."""
    if kind == "plrnn":
        c = W.random_plrnn_case(M, M, 1, 160, 0.2, 10 + M, w_norm=w_norm, a_range=(0.3, 0.75))
    else:
        c = W.random_shplrnn_case(M, L, M, 1, 160, 0.2, 10 + M, w_norm=w_norm, a_range=(0.3, 0.6))
    z = 3.0 * np.random.default_rng(M).standard_normal((1, 160, M)).astype(np.float32)
    return oracle_model(c), c.x[..., :1], z


@pytest.mark.parametrize("kind,M,L,w_norm", [("plrnn", 20, 0, 0.9), ("plrnn", 33, 0, 0.9), ("plrnn", 64, 0, 0.9),
                                             ("shplrnn", 5, 50, 4.0), ("shplrnn", 32, 64, 1.6), ("shplrnn", 64, 40, 2.2)])
def test_products_follow_the_masks(kind, M, L, w_norm):
    """Intermediate updates, where a product kept past a change of its masks would show (the fixed point
    would not: the residual and the chunks' re-run are exact)."""
    os.environ["DEER_CHUNK"] = "16"
    m, x, z = _stale_case(kind, M, L, w_norm)
    say("split masks", kind, M)
    for k in (2, 3):
        ref = _chunked_newton(m, x, 0.05, 1, z, 16, updates=k)[0]
        bad = _chunked_newton(m, x, 0.05, 1, z, 16, updates=k, stale="masks")[0]
        assert rel_inf(bad, ref) > 100 * TOL
        res = D.deer_solve(m, x, 0.05, 1, fixed_iters=k, init="user", z=torch.tensor(z, device="cuda"))
        assert rel_inf(res["z"].cpu().numpy(), ref) < TOL


@pytest.mark.parametrize("kind,M,L,w_norm,bound,passes", [
    ("plrnn", 20, 0, 1.1, 1.5, 3), ("plrnn", 64, 0, 0.9, 2.0, 3), ("shplrnn", 5, 50, 5.0, 10.0, 3),
    ("shplrnn", 32, 64, 2.2, 3.0, 4), ("shplrnn", 64, 40, 4.0, 3.0, 3)])
def test_products_follow_the_damping(kind, M, L, w_norm, bound, passes):
    """A rejected update is tried again at the same masks with another damping: the iterate after a few
    passes is that of products formed with it."""
    os.environ["DEER_CHUNK"] = "16"
    m, x, z = _stale_case(kind, M, L, w_norm)
    ref, accepted, gap = _chunked_newton(m, x, 0.05, 1, z, 16, passes=passes, bound=bound)
    bad = _chunked_newton(m, x, 0.05, 1, z, 16, passes=passes, bound=bound, stale="damping")[0]
    assert 0 < accepted < passes and gap > 0.05 and rel_inf(bad, ref) > 100 * TOL
    say("split damping", kind, M)
    res = D.deer_solve(m, x, 0.05, 1, tol=0.0, max_iter=passes, step_bound=bound, init="user",
                       z=torch.tensor(z, device="cuda"), check=False)
    assert res["status"] == 2 and res["iters"][0] == accepted
    assert rel_inf(res["z"].cpu().numpy(), ref) < TOL


def test_nonfinite_weights():
    c = _case(40, 40, 2, 64, 6300)
    m = oracle_model(c)
    m["W"] = m["W"].copy()
    m["W"][3, 5] = np.nan
    say("split NaN weights")
    assert D.deer_solve(m, c.x, 0.2, 40, tol=1e-5, max_iter=50)["status"] == 3


@pytest.mark.parametrize("M,N,B,T,chunk,T_w,own", [
    (17, 3, 2, 40, 5, 0, False), (20, 20, 1, 130, 65, 0, True), (32, 8, 17, 64, 16, 9, False), (33, 33, 2, 201, 66, 0, True),
    (48, 12, 3, 65, 8, 64, False), (64, 64, 2, 1, 16, 0, False), (64, 64, 3, 2, 1, 0, True), (64, 4, 2, 90, 31, 30, True),
    (64, 64, 1, 300, 100, 0, False)])
def test_adjoint(M, N, B, T, chunk, T_w, own):
    """lam and the gradients with the MSE seed and with a given cotangent and initial state, against
    the oracle at the same float32 trajectory."""
    os.environ["DEER_CHUNK"] = str(chunk)
    c = _case(M, N, B, T, 6400 + M + T)
    m = oracle_model(c)
    rng = np.random.default_rng(M)
    z0 = rng.standard_normal((B, M)).astype(np.float32) if own else None
    z32 = O.rollout(m, c.x, 0.2, N, z0=z0, T_w=T_w).astype(np.float32)
    g = rng.standard_normal(z32.shape).astype(np.float32) if own else None
    say("split adjoint", M, N, B, T, chunk, T_w, own)
    out = D.deer_adjoint(m, c.x, z32, 0.2, N, z0=z0, g=g, T_w=T_w)
    lam = O.adjoint(m, c.x, z32, 0.2, N, z0=z0, g=g, mask_precision="float32", T_w=T_w)
    ref = O.param_grads(m, c.x, z32, 0.2, N, lam, z0=z0, mask_precision="float32", T_w=T_w)
    assert rel_inf(out["lam"].cpu().numpy(), lam) < TOL
    for k in ("A", "W", "h"):
        assert rel_inf(out["grads"][k].cpu().numpy(), ref[k]) < TOL, k


@pytest.mark.parametrize("M", [32, 64])
def test_unaligned_rows(M):
    """x, z and g four bytes off a 16-byte boundary: the scalar loads give the values of the wide ones."""
    c = _case(M, M, 2, 150, 6500 + M)
    m = oracle_model(c)

    def off(t):
        b = torch.empty(t.numel() + 1, device="cuda")
        b[1:] = t.reshape(-1)
        return b[1:].view(t.shape)

    x = torch.from_numpy(c.x).cuda()
    g = torch.randn(2, 150, M, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    say("split unaligned", M)
    res = [D.deer_solve(m, xx, 0.2, M, tol=1e-5, z=zz) for xx, zz in ((x, torch.empty(2, 150, M, device="cuda")),
                                                                     (off(x), off(torch.empty(2, 150, M, device="cuda"))))]
    assert torch.equal(res[0]["z"], res[1]["z"])
    for gg in (None, g):
        a = D.deer_adjoint(m, x, res[0]["z"], 0.2, M, g=gg)
        b = D.deer_adjoint(m, off(x), off(res[0]["z"]), 0.2, M, g=None if gg is None else off(gg))
        assert torch.equal(a["lam"], b["lam"]) and all(torch.equal(a["grads"][k], b["grads"][k]) for k in a["grads"])


def _sh(M, L, N, B, T, seed, w_norm=0.3):
    return W.random_shplrnn_case(M, L, N, B, T, 0.2, seed, w_norm=w_norm, a_range=(0.3, 0.6))


# shallow model: widths and hidden counts at the edges of the tiles and of the 32-unit blocks (50 and
# 33 end inside one, 448 is about the largest), chunks shorter and longer than the steps formed together
@pytest.mark.parametrize("M,L,N,B,T,chunk,T_w", [
    (4, 50, 3, 2, 70, 9, 0), (16, 33, 5, 3, 64, 8, 20), (16, 448, 16, 1, 40, 16, 0), (17, 31, 3, 2, 33, 5, 0),
    (32, 256, 32, 2, 61, 20, 0), (20, 64, 8, 5, 50, 17, 49), (33, 128, 10, 2, 45, 10, 0), (64, 16, 64, 1, 90, 30, 11),
    (64, 128, 3, 2, 2, 1, 0), (5, 1, 2, 2, 30, 7, 0)])
def test_shallow_iterates_and_adjoint(M, L, N, B, T, chunk, T_w):
    os.environ["DEER_CHUNK"] = str(chunk)
    c = _sh(M, L, N, B, T, 6600 + M + L)
    m = oracle_model(c)
    rng = np.random.default_rng(M)
    z0 = rng.standard_normal((B, M)).astype(np.float32)
    say("split shallow", M, L, N, B, T, chunk, T_w)
    for k in (1, 3):
        res = D.deer_solve(m, c.x, 0.2, N, fixed_iters=k, z0=z0, T_w=T_w)
        ref = O.newton(m, c.x, 0.2, N, fixed_iters=k, z0=z0, T_w=T_w)
        assert rel_inf(res["z"].cpu().numpy(), ref["z"]) < TOL
    z32 = O.rollout(m, c.x, 0.2, N, z0=z0, T_w=T_w).astype(np.float32)
    g = rng.standard_normal(z32.shape).astype(np.float32)
    out = D.deer_adjoint(m, c.x, z32, 0.2, N, z0=z0, g=g, T_w=T_w)
    lam = O.adjoint(m, c.x, z32, 0.2, N, z0=z0, g=g, mask_precision="float32", T_w=T_w)
    assert rel_inf(out["lam"].cpu().numpy(), lam) < TOL


@pytest.mark.parametrize("M,L", [(6, 40), (32, 100), (64, 64)])
@pytest.mark.parametrize("kind", ["large", "tiny", "rows", "zero"])
def test_shallow_scales(M, L, kind):
    os.environ["DEER_CHUNK"] = "12"
    c = _sh(M, L, M, 2, 60, 6700 + M)
    p = {k: v.copy() for k, v in c.params.items()}
    if kind == "large":
        p["W1"] *= 64.0
    elif kind == "tiny":
        p["W1"] *= 1e-6
        p["A"] *= 1e-3
    elif kind == "rows":
        p["W1"] *= (2.0 ** -np.linspace(0, 18, M)).astype(np.float32)[:, None]
        p["W2"] *= (2.0 ** -np.linspace(0, 12, L)).astype(np.float32)[:, None]
    else:
        p["W1"] *= 0.0
        p["W2"] *= 0.0
        p["A"] *= 0.0
    m = {"kind": "shplrnn", **p}
    say("split shallow scales", M, L, kind)
    res = D.deer_solve(m, c.x, 0.2, M, fixed_iters=1, init="zero")
    ref = O.newton(m, c.x, 0.2, M, fixed_iters=1, init="zero")
    assert rel_inf(res["z"].cpu().numpy(), ref["z"]) < TOL


@pytest.mark.parametrize("M,L,bound", [(5, 50, 0.0), (32, 64, 0.05), (64, 40, 0.05)])
def test_shallow_kept_products(M, L, bound):
    os.environ["DEER_CHUNK"] = "16"
    c = _sh(M, L, M, 3, 300, 6800 + M)
    m = oracle_model(c)
    ref = O.rollout(m, c.x, 0.2, M)
    say("split shallow kept products", M, L, bound)
    res = D.deer_solve(m, c.x, 0.2, M, tol=1e-5, max_iter=5000, step_bound=bound)
    assert res["status"] == 0 and rel_inf(res["z"].cpu().numpy(), ref) < TOL
    more = D.deer_solve(m, c.x, 0.2, M, fixed_iters=8)
    assert rel_inf(more["z"].cpu().numpy(), ref) < 1e-5


@pytest.mark.parametrize("M", [17, 32, 33, 64])
@pytest.mark.parametrize("ncs", [1, 2, 5, 95, 96, 97, 129, 530])
def test_carry_levels(M, ncs):
    """Carries in one level (up to 95 chunks) and two (groups of 8, 16, 32; a last group of one chunk),
    both directions, through the bare dense scan in chunks of two steps."""
    os.environ["DEER_CHUNK"] = "2"
    T = 2 * ncs - 1
    rng = np.random.default_rng(M + ncs)
    J = (rng.standard_normal((2, T, M, M)) * 0.5 / np.sqrt(M)).astype(np.float32)
    b = rng.standard_normal((2, T, M)).astype(np.float32)
    say("split carry", M, ncs)
    for rev in (False, True):
        y = D.deer_scan(0, J, b, reverse=rev).cpu().numpy()
        ref = np.empty(b.shape)
        v = np.zeros((2, M))
        for t in (range(T - 1, -1, -1) if rev else range(T)):
            if rev:
                v = (np.einsum("bji,bj->bi", J[:, t + 1].astype(np.float64), v) if t + 1 < T else 0.0) + b[:, t]
            else:
                v = (np.einsum("bij,bj->bi", J[:, t].astype(np.float64), v) if t > 0 else 0.0) + b[:, t]
            ref[:, t] = v
        assert rel_inf(y, ref) < 1e-5


@pytest.mark.parametrize("B,T,M,H,No", [(1, 130, 63, 127, 1), (3, 43, 5, 33, 4), (2, 1100, 64, 128, 3)])
@pytest.mark.parametrize("kind", ["rows", "tiny", "large", "exact", "nan", "inf", "inf_weight"])
def test_readout_scales(B, T, M, H, No, kind):
    """Read-out: rows of very different size, weights far from one, rows without an error, and rows or
    weights that are not finite (they reach the loss, and no other row's cotangent)."""
    rng = np.random.default_rng(7000 + M)
    p = {"Wa": rng.standard_normal((H, M)) / np.sqrt(M), "ca": 0.1 * rng.standard_normal(H),
         "Wb": rng.standard_normal((No, H)) / np.sqrt(H), "cb": 0.1 * rng.standard_normal(No)}
    h = rng.standard_normal((B, T, M)) + 1j * rng.standard_normal((B, T, M))
    x = rng.standard_normal((B, T + 1, No))
    if kind == "rows":
        h *= 2.0 ** rng.integers(-20, 21, (B, T, 1))
    elif kind == "tiny":
        p["Wa"] *= 2.0 ** -60
        p["Wb"] *= 2.0 ** -30
        h *= 2.0 ** 40
    elif kind == "large":
        p["Wa"] *= 2.0 ** 50
        p["Wb"] *= 2.0 ** 20
        h *= 2.0 ** -60
    elif kind == "exact":
        h[:, ::3] = 0.0
        p["ca"] = -np.abs(p["ca"])           # no unit is on in those rows: y = cb = x there
        x[:, 1::3] = p["cb"].astype(np.float32)
    p = {k: v.astype(np.float32) for k, v in p.items()}
    h, x = h.astype(np.complex64), x.astype(np.float32)
    hg, pg = h.copy(), dict(p)
    if kind in ("nan", "inf"):
        hg[0, 5, 0] = np.nan if kind == "nan" else np.inf
    if kind == "inf_weight":
        pg["Wa"] = p["Wa"].copy()
        pg["Wa"][1, 2] = np.inf
    say("split readout", B, T, M, H, No, kind)
    out = D.deer_readout_loss(pg, torch.tensor(hg), x, want_masks=True)
    mk = out["masks"].cpu().numpy().view(np.uint32).reshape(B, T, -1)
    on = ((mk[..., :, None] >> np.arange(32, dtype=np.uint32)) & 1).astype(bool).reshape(B, T, -1)[..., :H]
    gg = out["g"].cpu().numpy()
    gr = {k: v.cpu().numpy() for k, v in out["grads"].items()}
    s = O.diag_ssm_readout_preactivation(p, h)
    if kind == "inf_weight":
        assert not np.isfinite(float(out["loss"].cpu()[0]))
        s = s[..., np.arange(H) != 1]
        assert np.array_equal((s > 0)[np.abs(s) > 1e-5], on[..., np.arange(H) != 1][np.abs(s) > 1e-5])
        return
    rows = np.ones((B, T), bool)
    rows[0, 5] = kind not in ("nan", "inf")
    # decisions: fp32 sums of M products are within 1e-5 of sum |Wa| |h| + |ca|
    band = 1e-5 * (np.abs(h.real.astype(np.float64)) @ np.abs(p["Wa"].astype(np.float64)).T + np.abs(p["ca"]))
    clear = (np.abs(s) > band) & rows[..., None]
    assert np.array_equal(on[clear], (s > 0)[clear])
    loss, g, ref = O.diag_ssm_loss_and_seed(p, h, x, mask=on)
    # g: the same bound carried through y, dy and dS (a row's own sizes only)
    y_err = (band * on) @ np.abs(p["Wb"]).T.astype(np.float64) + 1e-5 * (np.abs(np.maximum(s, 0)) @ np.abs(p["Wb"]).T
                                                                         + np.abs(p["cb"]) + np.abs(x[:, 1:]))
    tol = 2.0 / (B * No * T) * 2.0 * (y_err @ np.abs(p["Wb"]).astype(np.float64)) @ np.abs(p["Wa"]).astype(np.float64)
    assert (np.abs(gg - g) <= tol)[rows].all()
    if kind == "exact":
        assert not gg[:, ::3].any()
    if kind == "inf":
        assert not np.isfinite(float(out["loss"].cpu()[0]))
        return
    if kind == "nan":   # no unit is on in the row: y = cb, as for a row of zeros with every unit off
        assert not on[0, 5].any() and not gg[0, 5].any()
        assert np.isnan(gr["Wa"][:, 0]).all()
        gr["Wa"][:, 0] = ref["Wa"][:, 0]
    assert abs(float(out["loss"].cpu()[0]) - loss) <= 1e-5 * loss
    for k in ("Wa", "ca", "Wb", "cb"):
        assert rel_inf(gr[k], ref[k]) < TOL, k


@pytest.mark.parametrize("M,B,T,chunk", [(65, 1, 31, 3), (100, 2, 64, 4), (127, 1, 200, 2), (128, 1, 130, 2)])
@pytest.mark.parametrize("rev", [False, True])
@pytest.mark.parametrize("tr", [False, True])
@pytest.mark.parametrize("kind", ["plain", "rows", "small", "zero"])
def test_wide_scan_scales(M, B, T, chunk, rev, tr, kind):
    """Widths 65..128: all directions and orientations, with one and two carry levels, last chunks and
    groups of one, and rows of a matrix (or whole matrices) of very different size."""
    os.environ["DEER_CHUNK"] = str(chunk)
    rng = np.random.default_rng(7300 + M)
    J = rng.standard_normal((B, T, M, M)) * 0.6 / np.sqrt(M)
    if kind == "rows":
        J *= 2.0 ** -rng.integers(0, 24, (B, T, M, 1))
    elif kind == "small":
        J *= 2.0 ** -rng.integers(0, 60, (B, T, 1, 1))
    elif kind == "zero":
        J[:, 1::2] = 0.0
    J = J.astype(np.float32)
    b = rng.standard_normal((B, T, M)).astype(np.float32)
    say("split wide scan", M, B, T, chunk, rev, tr, kind)
    y = D.deer_scan(0, J, b, reverse=rev, transpose=tr).cpu().numpy()
    ref = np.empty(b.shape)
    v = np.zeros((B, M))
    Jd = J.astype(np.float64).transpose(0, 1, 3, 2) if tr else J.astype(np.float64)
    for t in (range(T - 1, -1, -1) if rev else range(T)):
        k = t + 1 if rev else t
        v = (np.matmul(Jd[:, k], v[..., None])[..., 0] if (0 < k < T) else 0.0) + b[:, t]
        ref[:, t] = v
    assert rel_inf(y, ref) < 1e-5
