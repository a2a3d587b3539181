"""Latents, hidden units and channels in units of their own.

A diagonal change of variables by powers of two is exact in float32, so a path whose operands, products
and sums keep float32's precision and range returns the same bits in the new units (times the units),
whatever the units' spread.  And matrices whose products are exact in float32 (24-bit entries times
powers of two) come out exact."""
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
SPREADS = [8, 24, 40]   # bits between the smallest and the largest unit


@pytest.fixture(autouse=True)
def _chunk():
    os.environ.pop("DEER_CHUNK", None)
    yield
    os.environ.pop("DEER_CHUNK", None)


def _units(n, bits, rng):
    """n powers of two over `bits` bits, permuted."""
    e = np.round(np.linspace(-bits / 2, bits / 2, n)).astype(int)
    return (2.0 ** rng.permutation(e)).astype(np.float32)


def _np(t):
    return t.cpu().numpy()


def _mant(n, rng):
    """n floats 1 + k 2^-23 with odd k: all 24 bits of the significand in use."""
    return (1.0 + (2.0 * rng.integers(1 << 18, 1 << 22, n) + 1.0) * 2.0 ** -23).astype(np.float32)


# ---- read-out of the diagonal SSM ---------------------------------------------------------------

def test_readout_decisions_to_the_last_bit():
    """s = h_0 - h_1 with h_0 the float after h_1: exact in float32, one unit in the last place above
    zero, so the hidden unit is on (and off the other way round)."""
    B, T, M, H = 2, 200, 64, 128
    rng = np.random.default_rng(1)
    p = {"Wa": np.zeros((H, M), np.float32), "ca": np.zeros(H, np.float32),
         "Wb": rng.standard_normal((3, H)).astype(np.float32), "cb": np.zeros(3, np.float32)}
    i, j = 2 * rng.integers(0, M // 2, H), 2 * rng.integers(0, M // 2, H) + 1
    p["Wa"][np.arange(H), i], p["Wa"][np.arange(H), j] = 1.0, -1.0
    lo = (rng.integers(1 << 23, (1 << 24) - 1, (B, T, 1)) + np.zeros((1, 1, M))).astype(np.float32)
    up = rng.random((B, T, M)) < 0.5
    h = np.where(up, np.nextafter(lo, np.float32(np.inf)), lo).astype(np.float32)
    x = rng.standard_normal((B, T + 1, 3)).astype(np.float32)
    say("units readout decisions")
    out = D.deer_readout_loss(p, torch.tensor(h.astype(np.complex64)), x, want_masks=True)
    mk = _np(out["masks"]).view(np.uint32).reshape(B, T, -1)
    on = ((mk[..., :, None] >> np.arange(32, dtype=np.uint32)) & 1).astype(bool).reshape(B, T, -1)[..., :H]
    assert np.array_equal(on, up[..., i] & ~up[..., j])


@pytest.mark.parametrize("bits", SPREADS)
@pytest.mark.parametrize("M,H", [(64, 128), (37, 50)])
def test_readout_channel_units(M, H, bits):
    B, T, K = 2, 1100, 3
    rng = np.random.default_rng(M)
    p = {"Wa": rng.standard_normal((H, M)) / np.sqrt(M), "ca": 0.1 * rng.standard_normal(H),
         "Wb": rng.standard_normal((K, H)) / np.sqrt(H), "cb": 0.1 * rng.standard_normal(K)}
    p = {k: v.astype(np.float32) for k, v in p.items()}
    h = (rng.standard_normal((B, T, M)) + 1j * rng.standard_normal((B, T, M))).astype(np.complex64)
    x = rng.standard_normal((B, T + 1, K)).astype(np.float32)
    d, e = _units(M, bits, rng), _units(H, bits, rng)
    q = {"Wa": e[:, None] * p["Wa"] / d, "ca": e * p["ca"], "Wb": p["Wb"] / e, "cb": p["cb"]}
    say("units readout", M, H, bits)
    a, b = D.deer_readout_loss(p, torch.tensor(h), x), D.deer_readout_loss(q, torch.tensor(h * d), x)
    assert torch.equal(a["loss"], b["loss"])
    assert np.array_equal(_np(a["g"]), _np(b["g"]) * d)
    for k, s in (("Wa", d[None, :] / e[:, None]), ("ca", 1 / e), ("Wb", e), ("cb", 1.0)):
        assert np.array_equal(_np(a["grads"][k]) * s, _np(b["grads"][k])), k


@pytest.mark.parametrize("bits", [12, 18])
def test_readout_rows_of_opposite_size(bits):
    """Large states where the error is small and small ones where it is large: every row counts alike
    in dWa.  Every unit is on with relu = 1, so y and the errors are exact."""
    B, T, M, H = 1, 640, 64, 128
    rng = np.random.default_rng(bits)
    p = {"Wa": np.zeros((H, M), np.float32), "ca": np.ones(H, np.float32),
         "Wb": (rng.integers(-3, 4, (2, H)) / 64).astype(np.float32), "cb": np.zeros(2, np.float32)}
    k = rng.integers(0, bits + 1, T)
    err = rng.integers(1, 4, (T, 2)) * rng.choice([-1.0, 1.0], (T, 2)) * 2.0 ** -k[:, None]
    x = np.zeros((B, T + 1, 2), np.float32)
    x[0, 1:] = p["Wb"].sum(1) - err
    h = (rng.standard_normal((B, T, M)) * 2.0 ** k[:, None]).astype(np.float32)
    say("units readout rows", bits)
    out = D.deer_readout_loss(p, torch.tensor(h.astype(np.complex64)), x)
    ref = O.diag_ssm_loss_and_seed(p, h.astype(np.complex64), x)[2]
    # fp32 sums of 640 terms of like size
    assert rel_inf(_np(out["grads"]["Wa"]), ref["Wa"]) < 1e-5


# ---- vanilla PLRNN, chunk products of 16 < M <= 64 ------------------------------------------------

@pytest.mark.parametrize("bits", SPREADS)
@pytest.mark.parametrize("M,N,T_w", [(20, 20, 0), (32, 8, 7), (64, 64, 0), (50, 3, 40)])
def test_vanilla_units(M, N, T_w, bits):
    """Newton iterates, lam and gradients."""
    os.environ["DEER_CHUNK"] = "12"
    B, T = 2, 150
    rng = np.random.default_rng(M)
    c = W.random_plrnn_case(M, N, B, T, 0.2, 900 + M, w_norm=0.4, a_range=(0.3, 0.8))
    p = c.params
    z0, g = rng.standard_normal((B, M)).astype(np.float32), rng.standard_normal((B, T, M)).astype(np.float32)
    d = _units(M, bits, rng)
    q = {"A": p["A"], "W": d[:, None] * p["W"] / d, "h": d * p["h"]}
    m, mu = oracle_model(c), {"kind": "plrnn", **q}
    say("units vanilla", M, N, T_w, bits)
    ref = O.newton(m, c.x, 0.2, N, fixed_iters=3, z0=z0, T_w=T_w)["z"]
    r = D.deer_solve(m, c.x, 0.2, N, fixed_iters=3, z0=z0, T_w=T_w)["z"]
    s = D.deer_solve(mu, c.x * d[:N], 0.2, N, fixed_iters=3, z0=z0 * d, T_w=T_w)["z"]
    assert rel_inf(_np(r), ref) < TOL
    assert np.array_equal(_np(r) * d, _np(s))
    a = D.deer_adjoint(m, c.x, r, 0.2, N, z0=z0, g=g, T_w=T_w)
    b = D.deer_adjoint(mu, c.x * d[:N], s, 0.2, N, z0=z0 * d, g=g / d, T_w=T_w)
    assert np.array_equal(_np(a["lam"]), _np(b["lam"]) * d)
    for k, u in (("A", 1.0), ("W", d[None, :] / d[:, None]), ("h", 1 / d)):
        assert np.array_equal(_np(a["grads"][k]) * u, _np(b["grads"][k])), k


def _one_on(B, T, M, rng):
    """States that are positive at one step of every latent, else negative; the adjoint of g = 2^e at the
    last step through J~ = diag(1 + w 1[z > 0]) is 2^e after that step and 2^e (1 + w) up to it."""
    t_on = rng.integers(0, T - 1, (B, M))
    z = np.where(np.arange(T)[None, :, None] == t_on[:, None, :], 1.0, -1.0).astype(np.float32)
    g = np.zeros((B, T, M), np.float32)
    g[:, -1] = 2.0 ** rng.integers(-3, 4, (B, M))

    def lam(full):
        return np.where(np.arange(T)[None, :, None] <= t_on[:, None, :], full, np.float32(1.0)) * g[:, -1:]
    return z, g, lam


@pytest.mark.parametrize("M", [20, 64])
def test_vanilla_products_keep_24_bits(M):
    os.environ["DEER_CHUNK"] = "16"
    B, T = 2, 200
    rng = np.random.default_rng(M)
    z, g, lam = _one_on(B, T, M, rng)
    full = _mant(M, rng)
    m = {"kind": "plrnn", "A": np.ones(M, np.float32), "W": np.diag(full - np.float32(1.0)), "h": np.zeros(M, np.float32)}
    say("units vanilla 24 bits", M)
    out = D.deer_adjoint(m, np.zeros((B, T + 1, 1), np.float32), z, 0.0, 1, g=g, z0=np.full((B, M), -1.0, np.float32))
    assert np.array_equal(_np(out["lam"]), lam(full))


# ---- shallow PLRNN ------------------------------------------------------------------------------------

@pytest.mark.parametrize("bits", SPREADS)
@pytest.mark.parametrize("M,L,N,T_w", [(5, 50, 3, 0), (32, 256, 32, 9), (64, 40, 10, 0), (100, 50, 3, 0), (67, 30, 20, 9)])
def test_shallow_units(M, L, N, T_w, bits):
    """Newton iterates, lam and gradients, latents and hidden units in units of their own (M > 64: the
    path that stores the Jacobians)."""
    os.environ["DEER_CHUNK"] = "12"
    B, T = 2, 90
    rng = np.random.default_rng(M)
    c = W.random_shplrnn_case(M, L, N, B, T, 0.2, 950 + M, w_norm=0.3, a_range=(0.3, 0.6))
    p = c.params
    z0, g = rng.standard_normal((B, M)).astype(np.float32), rng.standard_normal((B, T, M)).astype(np.float32)
    d, e = _units(M, bits, rng), _units(L, bits, rng)
    q = {"A": p["A"], "W1": d[:, None] * p["W1"] / e, "W2": e[:, None] * p["W2"] / d, "h1": d * p["h1"], "h2": e * p["h2"]}
    m, mu = oracle_model(c), {"kind": "shplrnn", **q}
    say("units shallow", M, L, N, T_w, bits)
    ref = O.newton(m, c.x, 0.2, N, fixed_iters=3, z0=z0, T_w=T_w)["z"]
    r = D.deer_solve(m, c.x, 0.2, N, fixed_iters=3, z0=z0, T_w=T_w)["z"]
    s = D.deer_solve(mu, c.x * d[:N], 0.2, N, fixed_iters=3, z0=z0 * d, T_w=T_w)["z"]
    assert rel_inf(_np(r), ref) < TOL
    assert np.array_equal(_np(r) * d, _np(s))
    a = D.deer_adjoint(m, c.x, r, 0.2, N, z0=z0, g=g, T_w=T_w)
    b = D.deer_adjoint(mu, c.x * d[:N], s, 0.2, N, z0=z0 * d, g=g / d, T_w=T_w)
    assert np.array_equal(_np(a["lam"]), _np(b["lam"]) * d)
    for k, u in (("A", 1.0), ("W1", e[None, :] / d[:, None]), ("W2", d[None, :] / e[:, None]), ("h1", 1 / d), ("h2", 1 / e)):
        assert np.array_equal(_np(a["grads"][k]) * u, _np(b["grads"][k])), k


@pytest.mark.parametrize("M,L", [(6, 10), (30, 40), (64, 64), (70, 64)])
def test_shallow_products_keep_24_bits(M, L):
    os.environ["DEER_CHUNK"] = "16"
    B, T = 2, 200
    rng = np.random.default_rng(M)
    z, g, lam = _one_on(B, T, M, rng)
    K = min(M, L)
    full = np.ones(M, np.float32)
    full[:K] = _mant(K, rng)
    W1, W2 = np.zeros((M, L), np.float32), np.zeros((L, M), np.float32)
    W1[np.arange(K), np.arange(K)] = 1.0
    W2[np.arange(K), np.arange(K)] = full[:K] - np.float32(1.0)
    m = {"kind": "shplrnn", "A": np.ones(M, np.float32), "W1": W1, "W2": W2, "h1": np.zeros(M, np.float32),
         "h2": np.zeros(L, np.float32)}
    say("units shallow 24 bits", M, L)
    out = D.deer_adjoint(m, np.zeros((B, T + 1, 1), np.float32), z, 0.0, 1, g=g, z0=np.full((B, M), -1.0, np.float32))
    assert np.array_equal(_np(out["lam"]), lam(full))


# ---- stored Jacobians, 64 < M <= 128 -------------------------------------------------------------------

@pytest.mark.parametrize("bits", SPREADS)
@pytest.mark.parametrize("M,L", [(65, 33), (100, 50), (128, 62)])
def test_wide_jacobian_units(M, L, bits):
    """J~ as the caller gets it."""
    B, T, N = 2, 40, 20
    rng = np.random.default_rng(M)
    c = W.random_shplrnn_case(M, L, N, B, T, 0.2, 970 + M, w_norm=0.3)
    p = c.params
    z = rng.standard_normal((B, T, M)).astype(np.float32)
    d, e = _units(M, bits, rng), _units(L, bits, rng)
    q = {"A": p["A"], "W1": d[:, None] * p["W1"] / e, "W2": e[:, None] * p["W2"] / d, "h1": d * p["h1"], "h2": e * p["h2"]}
    say("units wide jacobian", M, L, bits)
    a = D.plrnn_jacobian(oracle_model(c), c.x, z, 0.2, N, dense_J=True)
    b = D.plrnn_jacobian({"kind": "shplrnn", **q}, c.x * d[:N], z * d, 0.2, N, dense_J=True)
    assert torch.equal(a["masks"], b["masks"])
    assert np.array_equal(_np(a["J"]) * (d[:, None] / d), _np(b["J"]))


def test_wide_jacobian_keeps_24_bits():
    M, L, B, T = 128, 60, 1, 20
    rng = np.random.default_rng(3)
    z = rng.standard_normal((B, T, M)).astype(np.float32)
    W1, W2 = np.zeros((M, L), np.float32), np.zeros((L, M), np.float32)
    W1[2 * np.arange(L) + 1, np.arange(L)] = _mant(L, rng)
    W2[np.arange(L), 2 * np.arange(L)] = 2.0 ** rng.integers(-9, 10, L)
    m = {"kind": "shplrnn", "A": _mant(M, rng), "W1": W1, "W2": W2, "h1": np.zeros(M, np.float32),
         "h2": np.zeros(L, np.float32)}
    say("units wide jacobian 24 bits")
    J = _np(D.plrnn_jacobian(m, np.zeros((B, T + 1, 1), np.float32), z, 0.0, 1,
                             z0=rng.standard_normal((B, M)).astype(np.float32), dense_J=True)["J"])[:, 1:]
    on = z[:, :-1, 2 * np.arange(L)] > 0
    ref = np.zeros_like(J)
    ref[..., np.arange(M), np.arange(M)] = m["A"]
    ref[..., 2 * np.arange(L) + 1, 2 * np.arange(L)] = on * (W1[2 * np.arange(L) + 1, np.arange(L)]
                                                              * W2[np.arange(L), 2 * np.arange(L)])
    assert np.array_equal(J, ref)


@pytest.mark.parametrize("bits", SPREADS)
@pytest.mark.parametrize("rev", [False, True])
@pytest.mark.parametrize("tr", [False, True])
@pytest.mark.parametrize("M,B,T,chunk", [(30, 2, 70, 8), (65, 1, 31, 3), (128, 1, 130, 2), (100, 2, 64, 4)])
def test_scan_units(M, B, T, chunk, rev, tr, bits):
    """The bare scan, one and two carry levels, every step's state in its own units."""
    os.environ["DEER_CHUNK"] = str(chunk)
    rng = np.random.default_rng(M + T)
    J = (rng.standard_normal((B, T, M, M)) * 0.6 / np.sqrt(M)).astype(np.float32)
    b = rng.standard_normal((B, T, M)).astype(np.float32)
    d = np.stack([np.stack([_units(M, bits, rng) for _ in range(T)]) for _ in range(B)])
    # op(J_t) maps state t - 1 to t (reverse: t to t - 1)
    prev = np.concatenate([np.ones_like(d[:, :1]), d[:, :-1]], 1)
    out, inp = (prev, d) if rev else (d, prev)
    Jd = J * (inp[:, :, :, None] ** -1 * out[:, :, None, :] if tr else out[:, :, :, None] / inp[:, :, None, :])
    say("units scan", M, B, T, chunk, rev, tr, bits)
    y = _np(D.deer_scan(0, J, b, reverse=rev, transpose=tr))
    yd = _np(D.deer_scan(0, Jd.astype(np.float32), b * d, reverse=rev, transpose=tr))
    assert np.array_equal(y * d, yd)


@pytest.mark.parametrize("rev", [False, True])
@pytest.mark.parametrize("tr", [False, True])
@pytest.mark.parametrize("M,T,chunk", [(128, 64, 8), (70, 120, 2)])
def test_wide_scan_keeps_24_bits(M, T, chunk, rev, tr):
    """Permutations and one diagonal matrix of 24-bit entries: the scan of a state of powers of two is
    exact, through chunk products, group maps (two carry levels at T = 120) and carries."""
    os.environ["DEER_CHUNK"] = str(chunk)
    rng = np.random.default_rng(M)
    J = np.zeros((1, T, M, M), np.float32)
    for t in range(T):
        J[0, t, np.arange(M), rng.permutation(M)] = 1.0
    J[0, T // 2] = np.diag(_mant(M, rng))
    b = np.zeros((1, T, M), np.float32)
    b[0, T - 1 if rev else 0] = 2.0 ** rng.integers(-5, 6, M)
    say("units wide scan 24 bits", M, rev, tr)
    y = _np(D.deer_scan(0, J, b, reverse=rev, transpose=tr))[0]
    ref = np.zeros((T, M))
    v = np.zeros(M)
    for t in (range(T - 1, -1, -1) if rev else range(T)):
        k = t + 1 if rev else t
        if 0 < k < T:
            v = (J[0, k].T if tr else J[0, k]).astype(np.float64) @ v
        v = v + b[0, t]
        ref[t] = v
    assert np.array_equal(y, ref)
