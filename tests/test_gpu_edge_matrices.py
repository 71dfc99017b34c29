"""GPU parity of the degree-4 edge pass through per-edge matrices at the edges
of its tiles, against the oracle on sampled nodes (a hub whose segment spans
many ranges and nodes without edges among them).  The pass is taken from a
range per team of the device on, so the graphs have 50 to 70 thousand edges; that
it is taken is checked too.
Ranks just past a 32-rank tile and at the last one, channel counts with a part
tile, two, three, five and eight tiles, two and sixteen radial functions, odd
range lengths, both feature types, rows over 40 binary orders, weights far
from one common scale, forward, backward and attention.  The bounds are those of every other parity test: 1e-5
for fp32 problems (the two-part fp16 splits keep 22 bits, the sums are fp32),
2e-2 for bf16 ones (8 bits, rounded features and matrices)."""
import numpy as np
import pytest
import torch

import paper_2507_01131_amd as tdn
import workloads
from oracle import attention, layer
from tests._gpu_helpers import (check_rows, check_scaled, device_inputs, grad_vec_scale, random_factors, rel_err,
                                tol)

pytestmark = pytest.mark.gpu

HUB = 7  # (no node from N - 5 on has edges)


@pytest.fixture(autouse=True)
def _form():
    """Every edge pass of a test went through per-edge matrices (the form with a
    launch of its own for the factors)."""
    passes = ("cp_edge_fwd", "cp_edge_fwd_att", "cp_edge_bwd_src")
    tdn.timer_enable(True)
    for k in (*passes, "edge_factors"):
        tdn.timer_read(k, reset=True)
    yield
    tdn.timer_enable(False)
    n = [tdn.timer_read(k, reset=True)[1] for k in (*passes, "edge_factors")]
    assert n[3] == sum(n[:3]) > 0


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _problem(seed, N, E, C, R, n_radial, srt, dtype, wide=False):
    w = workloads.random_graph(seed, n_nodes=N, n_edges=E, L=4, C=C, R=R, feat_dtype=dtype)
    rng = np.random.default_rng(seed)
    w["n_radial"] = n_radial
    w["radial_w"] = (rng.standard_normal((n_radial, R)) / np.sqrt(n_radial)).astype(np.float32)
    ei = np.minimum(w["edge_index"], N - 6)
    ei[1, 1000:1400] = HUB
    ei[0, 2000:2500] = HUB
    if srt:
        o = np.argsort(ei[1], kind="stable")
        ei, w["edge_vec"], w["presorted"] = ei[:, o], w["edge_vec"][o], True
    w["edge_index"] = np.ascontiguousarray(ei)
    if wide:
        w["x"] = np.ldexp(w["x"], rng.integers(-20, 21, (N, 1, 1))).astype(np.float32)
        w["grad_out"] = np.ldexp(w["grad_out"], rng.integers(-20, 21, (N, 1, 1))).astype(np.float32)
    return w, random_factors(4, R, seed)


def _nodes(N, seed):
    return np.unique(np.concatenate([[0, HUB, N - 6, N - 1], np.random.default_rng(seed).integers(0, N, 12)]))


CASES = [
    # N, E, C, R, n_radial, sorted, dtype, wide
    (1500, 60001, 80, 65, 2, False, "f32", False), (1500, 60010, 96, 96, 16, True, "f32", False),
    (1500, 50023, 48, 97, 8, False, "f32", False), (1500, 50001, 128, 128, 9, False, "f32", True),
    (700, 60007, 160, 127, 8, False, "f32", False), (500, 50001, 256, 66, 8, True, "f32", False),
    (1500, 60003, 32, 128, 8, False, "bf16", False), (1500, 70001, 128, 97, 3, True, "bf16", False),
    (500, 60005, 144, 70, 8, False, "bf16", False), (500, 60001, 256, 128, 8, False, "bf16", False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"E{c[1]}C{c[2]}R{c[3]}q{c[4]}{c[6]}")
def test_forward_and_backward(case):
    w, (A, B, D) = _problem(900 + case[2], *case)
    inp = device_inputs(w, A, B, D)
    res = tdn.forward(inp["x"], inp["edge_vec"], inp["edge_index"], inp["A"], inp["B"], inp["D"], inp["W"],
                      inp["radial_w"], L=4, r_cut=w["r_cut"], edges_sorted=w["presorted"])
    gx, _, gv = tdn.backward(res, _t(w["grad_out"]))
    torch.cuda.synchronize()
    args = (w["x"], w["edge_index"], w["edge_vec"], A, B, D, w["W"], w["radial_w"], w["r_cut"], 4)
    t = tol(w)
    nodes = _nodes(w["N"], 1)
    ref = layer.forward_at_nodes(nodes, *args)
    out = res.out.cpu().numpy()
    assert rel_err(out[nodes], ref) < t
    check_rows(out[nodes], ref, t, "out")
    assert not out[w["N"] - 1].any()
    sel = np.nonzero(np.isin(w["edge_index"][0], nodes))[0]
    rx, _, rv = layer.backward(*args, w["grad_out"], perm=sel)
    assert rel_err(gx.cpu().numpy()[nodes], rx[nodes]) < t
    check_rows(gx.cpu().numpy()[nodes], rx[nodes], t, "grad_x")
    check_scaled(gv.cpu().numpy()[sel], rv[sel], grad_vec_scale(w, A, B, D, edges=sel), t, "grad_edge_vec")
    assert np.all(np.isfinite(out)) and bool(torch.isfinite(gx).all())


def _ldexp(a, e):
    return np.ldexp(a, e).astype(np.float32)


def _weights(kind, w, f, rng):
    """Factors and radial weights (f: A, B, D) far from one common scale, the
    products of what they multiply near it."""
    A, B, D = f
    R, k = A.shape[1], np.arange(25)[:, None]
    if kind == "far":  # the largest radial weights at a distance that no edge has
        n = np.linalg.norm(w["edge_vec"], axis=1, keepdims=True)
        w["edge_vec"] = (w["edge_vec"] / n * (3.5 + 2.5 * rng.random(n.shape))).astype(np.float32)
        w["radial_w"][0] *= 1e5
    elif kind == "ranks":
        e = rng.integers(-10, 11, (3, R))
        A, B, D, w["radial_w"] = _ldexp(A, e[0]), _ldexp(B, e[1]), _ldexp(D, e[2]), _ldexp(w["radial_w"], -e.sum(0))
    elif kind == "rank0":  # one rank's share of g
        B, D = B.copy(), D.copy()
        B[:, 0] *= 2.0 ** 20
        D[:, 0] *= 2.0 ** -20
    elif kind in ("small", "large"):  # B's squares below and above what fp32 holds
        s = {"small": -90, "large": 70}[kind]
        B, D = _ldexp(B, s), _ldexp(D, -s)
    elif kind == "rows":
        D = _ldexp(D, -(k % 5) * 3)
        A, w["x"] = _ldexp(A, -((k + 2) % 5) * 3), _ldexp(w["x"], ((k + 2) % 5) * 3)
    elif kind == "blocks":  # two groups of rows that share no rank, one of them with a small g
        keep = (np.arange(R)[None] < R // 2) == (k < 12)
        A, D = A * keep, D * keep
        B = B.copy()
        B[:, R // 2:] *= 2.0 ** -16
    elif kind == "axis":  # every edge where the first ranks' harmonic vanishes, the others' g small
        n = np.linalg.norm(w["edge_vec"], axis=1)
        w["edge_vec"] = np.stack([0 * n, 0 * n, np.where(np.arange(n.size) % 2, n, -n)], 1).astype(np.float32)
        B = np.where((k == 3) & (np.arange(R) < R // 2), B, 0) + np.where((k == 0) & (np.arange(R) >= R // 2),
                                                                         _ldexp(B, -40), 0)
        B = B.astype(np.float32)
    return A, B, D


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["far", "ranks", "rank0", "small", "large", "rows", "blocks", "axis"])
def test_weights_of_wide_range(kind, dtype):
    """The bounds per row of output and per degree row of it; a rank's, a row's
    or an edge's own scale must not show in them."""
    w, f = _problem(970, 700, 50013, 128, 120, 8, True, dtype)
    A, B, D = _weights(kind, w, f, np.random.default_rng(5))
    if dtype == "bf16":
        w["x_bf16"] = workloads.bf16_round(w["x"])
    inp = device_inputs(w, A, B, D)
    res = tdn.forward(inp["x"], inp["edge_vec"], inp["edge_index"], inp["A"], inp["B"], inp["D"], inp["W"],
                      inp["radial_w"], L=4, r_cut=w["r_cut"], edges_sorted=True)
    gx, _, _ = tdn.backward(res, _t(w["grad_out"]))
    torch.cuda.synchronize()
    args = (w["x"], w["edge_index"], w["edge_vec"], A, B, D, w["W"], w["radial_w"], w["r_cut"], 4)
    t = tol(w)
    nodes = _nodes(w["N"], 4)
    ref = layer.forward_at_nodes(nodes, *args)
    out = res.out.cpu().numpy()[nodes]
    assert rel_err(out, ref) < t
    check_rows(out.reshape(-1, 128), ref.reshape(-1, 128), t, "out")
    sel = np.nonzero(np.isin(w["edge_index"][0], nodes))[0]
    rx, _, _ = layer.backward(*args, w["grad_out"], perm=sel)
    gx = gx.cpu().numpy()[nodes]
    assert rel_err(gx, rx[nodes]) < t
    check_rows(gx.reshape(-1, 128), rx[nodes].reshape(-1, 128), t, "grad_x")


def test_radial_basis_far_from_its_centre():
    """One narrow radial function, 3 to 3.5 widths from its centre 13 sigma,
    sigma = 0.4: rounding the centre to fp32 by itself would be 2e-6 of the
    function.  Along the axes lengths are exact, and what the function has left is
    two roundings of (r - mu) / sigma, 3e-7 of it in the norm; the layer adds at
    most 6.2e-7 (its splits and sums)."""
    w, f = _problem(972, 700, 50013, 64, 128, 16, True, "f32")
    rng = np.random.default_rng(6)
    w["r_cut"] = 6.0
    vec = np.zeros((w["E"], 3), np.float32)
    vec[np.arange(w["E"]), rng.integers(0, 3, w["E"])] = 3.8 + 0.2 * rng.random(w["E"])
    w["edge_vec"] = vec * rng.choice([-1.0, 1.0], (w["E"], 1)).astype(np.float32)
    w["radial_w"][np.arange(16) != 13] = 0.0
    inp = device_inputs(w, *f)
    res = tdn.forward(inp["x"], inp["edge_vec"], inp["edge_index"], inp["A"], inp["B"], inp["D"], inp["W"],
                      inp["radial_w"], L=4, r_cut=6.0, edges_sorted=True)
    nodes = _nodes(w["N"], 4)
    ref = layer.forward_at_nodes(nodes, w["x"], w["edge_index"], w["edge_vec"], *f, w["W"], w["radial_w"], 6.0, 4)
    assert rel_err(res.out.cpu().numpy()[nodes], ref) < 1e-6


def test_infinity_stays_in_its_row():
    w, (A, B, D) = _problem(971, 700, 50013, 64, 100, 8, True, "f32")
    clean = D.copy()
    D[3, 5], clean[3] = np.inf, 0.0
    inp = device_inputs(w, A, B, D)
    res = tdn.forward(inp["x"], inp["edge_vec"], inp["edge_index"], inp["A"], inp["B"], inp["D"], inp["W"],
                      inp["radial_w"], L=4, r_cut=w["r_cut"], edges_sorted=True)
    nodes = _nodes(w["N"], 4)
    ref = layer.forward_at_nodes(nodes, w["x"], w["edge_index"], w["edge_vec"], A, B, clean, w["W"], w["radial_w"],
                                 w["r_cut"], 4)
    out, rest = res.out.cpu().numpy()[nodes], np.arange(25) != 3
    assert not np.isfinite(out[0, 3]).any()
    check_rows(out[:, rest], ref[:, rest], tol(w), "out")


@pytest.mark.parametrize("N,E,C,R,H", [(1500, 60003, 96, 65, 3), (1500, 50001, 128, 128, 4), (500, 60002, 256, 97, 8)])
def test_attention(N, E, C, R, H):
    w, (A, B, D) = _problem(950 + C, N, E, C, R, 8, False, "f32")
    rng = np.random.default_rng(E)
    W1 = (2 * rng.standard_normal((2 * C + 8, 16)) / np.sqrt(2 * C + 8)).astype(np.float32)
    w2 = (rng.standard_normal((16, H)) / 2).astype(np.float32)
    res, _ = tdn.attention_forward(_t(w["x"]), _t(w["edge_vec"]), _t(w["edge_index"]), _t(A), _t(B), _t(D),
                                   _t(w["W"]), _t(w["radial_w"]), _t(W1), _t(w2), L=4, r_cut=w["r_cut"],
                                   edges_sorted=False)
    torch.cuda.synchronize()
    nodes = _nodes(N, 2)
    perm, _ = layer.stable_sort_by_key(w["edge_index"][1], N)
    sub = perm[np.isin(w["edge_index"][1][perm], nodes)]
    ref, _ = attention.forward(w["x"], w["edge_index"], w["edge_vec"], A, B, D, w["W"], w["radial_w"], W1, w2,
                               w["r_cut"], 4, perm=sub)
    out = res.out.cpu().numpy()
    assert np.all(np.isfinite(out))
    assert rel_err(out[nodes], ref[nodes]) < tol(w)
    check_rows(out[nodes], ref[nodes], tol(w), "out")
