"""GPU parity: RNN hot path (build_jacobians, scan, param_grads) through the C ABI
against the fp64 oracle, element by element on the same seeded inputs."""
import numpy as np
import pytest

import workloads
from oracle import rnn as orn
from oracle import scan as oscan
from util import TOL, per_step_err, rel_err, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1907_10134_amd as lib
    return lib


def _gpu_forward(bp, w):
    import torch
    T, B, H = w["T"], w["B"], w["H"]
    h = torch.zeros((T + 1, B, H), dtype=torch.float32, device="cuda")
    bp.forward(bp.RNN_TANH, to_gpu(w["x"]), to_gpu(w["w_ih"]), to_gpu(w["w_hh"]), to_gpu(w["b"]), None, h)
    return h


@pytest.mark.parametrize("T,B,H,I", [(16, 2, 20, 1), (5, 3, 7, 2), (33, 1, 32, 3), (9, 2, 1, 1)])
def test_forward_and_head_match_oracle(bp, T, B, H, I):
    w = workloads.rnn_inputs(T, B, H, I, 10, seed=3)
    h = _gpu_forward(bp, w)
    h_ref = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"])
    assert rel_err(to_np(h), h_ref) <= 1e-5
    seed, loss = bp.head_seed(h[-1].contiguous(), to_gpu(w["w_out"]), to_gpu(w["b_out"]), to_gpu(w["labels"]))
    l_ref, s_ref = orn.head(to_np(h[-1]), w["w_out"], w["b_out"], w["labels"])
    assert rel_err(to_np(seed), s_ref) <= 1e-5
    assert abs(float(loss.item()) - l_ref) <= 1e-5 * abs(l_ref)


@pytest.mark.parametrize("T,B,H", [(16, 2, 20), (3, 1, 1), (7, 3, 2), (5, 2, 16), (4, 2, 32),
                                   (130, 5, 20), (2, 2, 33), (2, 1, 128)])
def test_build_jacobians_rnn(bp, T, B, H):
    w = workloads.rnn_inputs(T, B, H, 1, 10, seed=T + H)
    h32 = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"]).astype(np.float32)
    Jt = bp.build_jacobians(bp.RNN_TANH, to_gpu(h32), w_hh=to_gpu(w["w_hh"]))
    ref = orn.jacobians_T(h32, w["w_hh"])
    assert rel_err(to_np(Jt), ref) <= 1e-6


SCAN_SHAPES = [(1, 2, 20), (2, 2, 20), (3, 1, 5), (63, 2, 20), (64, 2, 20), (65, 3, 20), (66, 1, 20),
               (127, 2, 16), (128, 2, 20), (129, 2, 20), (130, 16, 20), (200, 2, 32), (257, 3, 1),
               (300, 2, 2), (70, 2, 33), (131, 1, 64), (67, 2, 128), (1000, 16, 20), (4300, 2, 20),
               (200, 2, 128), (257, 3, 128), (130, 1, 128), (193, 2, 128),
               (1, 8, 20), (2, 16, 20), (33, 8, 20), (34, 24, 20), (97, 40, 20), (700, 32, 20),
               (150, 12, 20), (100, 6, 20), (90, 9, 20), (1100, 10, 20)]


@pytest.mark.parametrize("T,B,H", SCAN_SHAPES)
@pytest.mark.parametrize("want_g0", [False, True])
def test_scan_matches_linear_scan(bp, T, B, H, want_g0):
    import torch
    if T >= 1000:
        jt, seed = workloads.reflection_jacobian_chain(T, B, H, seed=T * 131 + H)
    else:
        jt, seed = workloads.random_jacobian_chain(T, B, H, seed=T * 131 + H, scale=1.05 / np.sqrt(H))
    G_ref, g0_ref = oscan.linear_scan(jt, seed)
    g0 = torch.empty((B, H), dtype=torch.float32, device="cuda") if want_g0 else None
    G = bp.scan(to_gpu(jt), to_gpu(seed), g0=g0)
    if H == 20:
        bp.check_scan()                 # synchronises; raises if a bounded wait inside the scan expired
    torch.cuda.synchronize()
    assert rel_err(to_np(G), G_ref) <= TOL
    assert per_step_err(to_np(G), G_ref) <= 2 * TOL
    assert np.array_equal(to_np(G[T - 1]), seed)
    if want_g0:
        assert rel_err(to_np(g0), g0_ref) <= TOL * max(1.0, np.max(np.abs(G_ref)) / np.max(np.abs(g0_ref)))


def test_scan_does_not_modify_inputs_and_is_repeatable(bp):
    import torch
    jt, seed = workloads.random_jacobian_chain(333, 4, 20, seed=9)
    djt, dseed = to_gpu(jt), to_gpu(seed)
    G1 = to_np(bp.scan(djt, dseed))
    G2 = to_np(bp.scan(djt, dseed))
    assert np.array_equal(to_np(djt), jt) and np.array_equal(to_np(dseed), seed)
    assert np.array_equal(G1, G2)


def test_scan_identity_and_diagonal_special_cases(bp):
    T, B, H = 150, 2, 20
    eye = np.broadcast_to(np.eye(H, dtype=np.float32), (T, B, H, H)).copy()
    seed = np.random.default_rng(0).standard_normal((B, H)).astype(np.float32)
    G = to_np(bp.scan(to_gpu(eye), to_gpu(seed)))
    assert all(np.array_equal(G[t], seed) for t in range(T))
    d = np.random.default_rng(1).uniform(0.9, 1.1, size=(T, B, H)).astype(np.float32)
    jt = np.zeros((T, B, H, H), np.float32)
    jt[..., np.arange(H), np.arange(H)] = d
    G = to_np(bp.scan(to_gpu(jt), to_gpu(seed)))
    cp = np.cumprod(d.astype(np.float64)[::-1], axis=0)[::-1]
    for t in range(1, T):
        assert np.allclose(G[t - 1], seed * cp[t], rtol=1e-4)


@pytest.mark.parametrize("T,B,H", [(150, 2, 1), (151, 3, 4), (90, 1, 12), (120, 2, 15), (300, 2, 16), (200, 5, 17), (140, 3, 31),
                                   (260, 40, 32), (130, 2, 36), (110, 3, 47), (230, 9, 48), (100, 2, 63), (170, 30, 64),
                                   (90, 2, 65), (140, 1, 80), (200, 7, 96), (80, 2, 100), (75, 1, 112), (70, 2, 113), (60, 1, 127),
                                   (40, 260, 8)])
def test_scan_of_general_sizes_in_segments(bp, T, B, H):
    """The kernels for every H without one of its own, around the multiples of 4 and 16 they round to:
    cut as the cost model does it with the workspace of the query, within the library's fixed scratch,
    and with the least workspace a call accepts (none for short chains)."""
    import torch
    jt, seed = workloads.random_jacobian_chain(T, B, H, seed=T * 7 + H, scale=1.05 / np.sqrt(H))
    G_ref, g0_ref = oscan.linear_scan(jt, seed)
    djt, dseed = to_gpu(jt), to_gpu(seed)
    g0 = torch.empty((B, H), dtype=torch.float32, device="cuda")
    G = bp.scan(djt, dseed, g0=g0)
    assert rel_err(to_np(G), G_ref) <= TOL and per_step_err(to_np(G), G_ref) <= 2 * TOL
    assert rel_err(to_np(g0), g0_ref) <= TOL
    G2 = torch.zeros_like(G)
    if T <= 64:
        code = bp.binding._lib.bppsa_scan(T, B, H, djt.data_ptr(), dseed.data_ptr(), G2.data_ptr(), None, None, 0, None)
        assert code == 0
    else:
        bp.scan_static(djt, dseed, G2)
    torch.cuda.synchronize()
    assert rel_err(to_np(G2), G_ref) <= TOL and per_step_err(to_np(G2), G_ref) <= 2 * TOL


@pytest.mark.parametrize("T,B,H,I", [(16, 2, 20, 1), (1, 1, 1, 1), (37, 3, 7, 2), (1000, 16, 20, 1),
                                     (40, 2, 32, 3), (9, 2, 64, 1)])
def test_param_grads_rnn(bp, T, B, H, I):
    w = workloads.rnn_inputs(T, B, H, I, 10, seed=T)
    h = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"])
    _, seed = orn.head(h[-1], w["w_out"], w["b_out"], w["labels"])
    G, _ = orn.backward_chain(h, w["w_hh"], seed)
    h32, G32 = h.astype(np.float32), G.astype(np.float32)
    ref = orn.param_grads(h32, w["x"], G32)
    dW_ih, dW_hh, db, db2 = bp.param_grads(bp.RNN_TANH, to_gpu(h32), to_gpu(w["x"]), to_gpu(G32))
    assert rel_err(to_np(dW_ih), ref[0]) <= TOL
    assert rel_err(to_np(dW_hh), ref[1]) <= TOL
    assert rel_err(to_np(db), ref[2]) <= TOL
    assert np.array_equal(to_np(db), to_np(db2))


@pytest.mark.parametrize("T,B,H,I", [(3, 11, 5, 1), (70, 3, 33, 17), (9, 7, 100, 1), (2100, 33, 16, 2), (65, 1, 127, 1),
                                     (40, 2, 1, 400), (21, 3, 33, 445)])
def test_param_grads_any_size(bp, T, B, H, I):
    """One output tile to ninety, a part of one in either direction, more inputs than threads, rows that end inside
    a tile of 32 and 69300 of them; h starts at an odd float."""
    import torch
    rng = np.random.default_rng(H)
    h = np.tanh(rng.standard_normal((T + 1, B, H))).astype(np.float32)
    G, x = rng.standard_normal((T, B, H)).astype(np.float32), rng.standard_normal((T, B, I)).astype(np.float32)
    ref = orn.param_grads(h, x, G)
    shifted = torch.full((h.size + 1 + 32 * H,), float("nan"), dtype=torch.float32, device="cuda")
    shifted[1:h.size + 1] = to_gpu(h).reshape(-1)
    got = bp.param_grads(bp.RNN_TANH, shifted[1:h.size + 1].reshape(h.shape), to_gpu(x), to_gpu(G))
    for k in range(3):
        assert rel_err(to_np(got[k]), ref[k]) <= TOL


@pytest.mark.parametrize("T,B,H", [(3, 5, 1), (40, 7, 5), (9, 3, 8), (2100, 1, 33), (300, 7, 64), (11, 2, 100), (2, 3, 130)])
def test_build_jacobians_any_size(bp, T, B, H):
    """Tiles of less than a workgroup's pieces, a stretch, and several with a part of one; every tile is written."""
    import torch
    rng = np.random.default_rng(H)
    h = np.tanh(rng.standard_normal((T + 1, B, H))).astype(np.float32)
    w = rng.standard_normal((H, H)).astype(np.float32)
    shifted = torch.empty(h.size + 1, dtype=torch.float32, device="cuda")
    shifted[1:] = to_gpu(h).reshape(-1)
    Jt = torch.full((T, B, H, H), float("nan"), dtype=torch.float32, device="cuda")
    bp.build_jacobians(bp.RNN_TANH, shifted[1:].reshape(h.shape), w_hh=to_gpu(w), Jt=Jt)
    h64, w64 = h[1:].astype(np.float64), w.astype(np.float64)
    ref = w64.T[None, None] * (1.0 - h64 * h64)[:, :, None, :]
    # two roundings of each entry
    assert np.all(np.abs(to_np(Jt) - ref) <= 2.0 ** -22 * np.abs(ref) + 1e-30)


@pytest.mark.parametrize("T,B", [(83887, 1), (10491, 8), (6001, 14), (400, 211), (5003, 17)])
def test_h20_jacobians_larger_than_the_caches(bp, T, B):
    """From 134 MB on (83887 tiles are the first) tiles are written and read past the caches.  The builder against its
    formula in 64 bits; the scan, in units on one die (8, 14) and at device scope (1, 17) and as a chain (211), gives the
    bits of the scan that forms the tiles itself."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(T)
    h = torch.rand((T + 1, B, 20), generator=g, device="cuda") * 1.2 - 0.6
    w = torch.linalg.qr(torch.randn((20, 20), generator=g, device="cuda"))[0].contiguous() * 1.1
    seed = torch.randn((B, 20), generator=g, device="cuda")
    Jt = torch.full((T, B, 20, 20), float("nan"), device="cuda")
    bp.build_jacobians(bp.RNN_TANH, h, w_hh=w, Jt=Jt)
    step = max(1, T // 50)
    ref = w.double().t()[None, None] * (1.0 - h[1:].double() ** 2)[::step, :, None, :]
    assert bool(torch.isfinite(Jt).all())
    assert float((Jt[::step].double() - ref).abs().max()) <= 4 * 2.0 ** -24 * 1.1     # one rounding of 1 - h^2, one of the product
    G, Gf = torch.empty((T, B, 20), device="cuda"), torch.empty((T, B, 20), device="cuda")
    bp.scan(Jt, seed, G)
    bp.check_scan()
    bp.rnn_scan_fused(h, w, seed, Gf)
    bp.check_scan()
    assert bool(torch.equal(G, Gf))


@pytest.mark.parametrize("T,B,I", [(63, 1, 3), (13, 5, 2), (129, 1, 1), (5003, 14, 1)])
def test_param_grads_h20_tile_edges(bp, T, B, I):
    """Rows that end one before, one past and inside a tile of 64, and workgroups of two tiles with the last ones
    empty (70042 rows); the rows behind the end of every array hold what must not be read into the sums."""
    rng = np.random.default_rng(T)
    H = 20
    h = np.tanh(rng.standard_normal((T + 1, B, H))).astype(np.float32)
    G, x = rng.standard_normal((T, B, H)).astype(np.float32), rng.standard_normal((T, B, I)).astype(np.float32)
    ref = orn.param_grads(h, x, G)

    def padded(a):
        import torch
        t = torch.full((a.size + 64 * H,), float("nan"), dtype=torch.float32, device="cuda")
        t[:a.size] = to_gpu(a).reshape(-1)
        return t[:a.size].reshape(a.shape)

    got = bp.param_grads(bp.RNN_TANH, padded(h), padded(x), padded(G))
    for k in range(3):
        assert rel_err(to_np(got[k]), ref[k]) <= TOL


def _end_to_end(bp, w, h32=None):
    """forward -> seed -> build_jacobians -> scan -> param_grads, all on the GPU.

    With h32 given, the hidden states are an input (the same fp32 values the oracle uses).
    """
    import torch
    h = _gpu_forward(bp, w) if h32 is None else to_gpu(h32)
    seed, _ = bp.head_seed(h[-1].contiguous(), to_gpu(w["w_out"]), to_gpu(w["b_out"]), to_gpu(w["labels"]))
    Jt = bp.build_jacobians(bp.RNN_TANH, h, w_hh=to_gpu(w["w_hh"]))
    g0 = torch.empty((w["B"], w["H"]), dtype=torch.float32, device="cuda")
    G = bp.scan(Jt, seed, g0=g0)
    grads = bp.param_grads(bp.RNN_TANH, h, to_gpu(w["x"]), G)
    torch.cuda.synchronize()
    if w["H"] == 20:
        bp.check_scan()
    return to_np(G), to_np(g0), [to_np(g) for g in grads]


def _oracle_end_to_end(w, h32=None):
    h = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"]) if h32 is None else h32
    _, seed = orn.head(h[-1], w["w_out"], w["b_out"], w["labels"])
    G, g0 = orn.backward_chain(h, w["w_hh"], seed)
    return G, g0, orn.param_grads(h, w["x"], G)


@pytest.mark.parametrize("cfg", [0, 1, 2])
def test_end_to_end_configs(bp, cfg):
    w = workloads.config_inputs(cfg)
    G, g0, grads = _end_to_end(bp, w)
    G_ref, g0_ref, grads_ref = _oracle_end_to_end(w)
    assert rel_err(G, G_ref) <= TOL
    for got, ref in zip(grads[:3], grads_ref):
        assert rel_err(got, ref) <= TOL
    # stricter, per time step, wherever the gradient has not underflowed fp32
    assert per_step_err(G, G_ref, floor=1e-30) <= 2 * TOL


@pytest.mark.parametrize("T", [1000, 30000])
def test_end_to_end_norm_preserving(bp, T):
    # gradients stay O(1) over the whole sequence, so every time step is a real comparison
    # (gain 1.1 sits at the edge of chaos, so the forward pass is taken from the oracle and
    # rounded once: both sides then start from identical fp32 hidden states)
    w = workloads.rnn_inputs_norm_preserving(T, 16, gain=1.02 if T == 1000 else 1.1)
    h32 = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"]).astype(np.float32)
    G, g0, grads = _end_to_end(bp, w, h32)
    G_ref, g0_ref, grads_ref = _oracle_end_to_end(w, h32)
    n = np.max(np.abs(G_ref.reshape(T, -1)), axis=1)
    assert n.min() > 1e-4 * n.max(), "test weights let the gradient vanish"
    assert rel_err(G, G_ref) <= TOL
    assert per_step_err(G, G_ref) <= 2 * TOL
    for got, ref in zip(grads[:3], grads_ref):
        assert rel_err(got, ref) <= TOL


def _ws(bp, T, B, H=20, fill=0xC3):
    import torch
    return torch.full((bp.scan_workspace_bytes(T, B, H),), fill, dtype=torch.uint8, device="cuda")


def _error_word(ws):
    import torch
    return int(ws[:4].view(torch.int32).item())


@pytest.mark.parametrize("T,B,H", [s for s in SCAN_SHAPES if s[2] == 20] +
                         [(2500, 16, 20), (64, 8, 20), (129, 8, 20), (2049, 3, 20), (5000, 8, 20), (3000, 12, 20)])
@pytest.mark.parametrize("want_g0", [False, True])
def test_scan_h20_units_of_two_halves_match_linear_scan(bp, T, B, H, want_g0):
    """The form of the H=20 scan that long chains take (units of 64 steps, the first half parked
    in registers), forced on every shape: chain lengths around multiples of 32 and 64, one unit
    only, batch sizes on and off the die-local path."""
    import torch
    if T >= 1000:
        jt, seed = workloads.reflection_jacobian_chain(T, B, H, seed=T * 131 + H)
    else:
        jt, seed = workloads.random_jacobian_chain(T, B, H, seed=T * 131 + H, scale=1.05 / np.sqrt(H))
    G_ref, g0_ref = oscan.linear_scan(jt, seed)
    g0 = torch.empty((B, H), dtype=torch.float32, device="cuda") if want_g0 else None
    ws = _ws(bp, T, B)
    G = bp.scan_h20_diag(to_gpu(jt), to_gpu(seed), g0=g0, workspace=ws, unit_halves=2)
    torch.cuda.synchronize()
    assert _error_word(ws) == 0
    assert rel_err(to_np(G), G_ref) <= TOL
    assert per_step_err(to_np(G), G_ref) <= 2 * TOL
    assert np.array_equal(to_np(G[T - 1]), seed)
    if want_g0:
        assert rel_err(to_np(g0), g0_ref) <= TOL * max(1.0, np.max(np.abs(G_ref)) / np.max(np.abs(g0_ref)))


@pytest.mark.parametrize("halves", [1, 2])
@pytest.mark.parametrize("mask", [0x01, 0xA5, 0xFF])
def test_scan_h20_fallback_when_dies_stand_aside(bp, mask, halves):
    """Chains whose compute die takes no part are picked up by the last workgroup (device-scope path)."""
    import torch
    T, B, H = 200, 16, 20
    jt, seed = workloads.random_jacobian_chain(T, B, H, seed=77, scale=1.05 / np.sqrt(H))
    G_ref, _ = oscan.linear_scan(jt, seed)
    djt, dseed = to_gpu(jt), to_gpu(seed)
    ws0 = _ws(bp, T, B)
    G_normal = to_np(bp.scan_h20_diag(djt, dseed, workspace=ws0, unit_halves=halves))
    ws = _ws(bp, T, B, fill=0)
    G = to_np(bp.scan_h20_diag(djt, dseed, workspace=ws, absent_dies=mask, unit_halves=halves))
    torch.cuda.synchronize()
    assert _error_word(ws0) == 0 and _error_word(ws) == 0     # no bounded wait expired
    assert rel_err(G, G_ref) <= TOL
    assert np.array_equal(G, G_normal)                        # same bits as the die-local path


@pytest.mark.parametrize("T,B,want_g0", [(1, 2, False), (1, 2, True), (16, 2, True), (33, 8, False), (130, 5, True),
                                         (1000, 16, False), (2100, 16, True)])
def test_rnn_scan_fused_matches_two_call_path_and_oracle(bp, T, B, want_g0):
    """bppsa_rnn_scan_fused: same bits as build_jacobians + scan, and the oracle's gradients."""
    import torch
    H = 20
    w = workloads.rnn_inputs_norm_preserving(T, B, seed=T + B, gain=1.05) if T >= 1000 else workloads.rnn_inputs(T, B, H, 1, 10, seed=T)
    h64 = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"])
    h32 = np.asarray(h64, np.float32)              # both sides start from the same fp32 states
    _, seed = orn.head(h32[-1].astype(np.float64), w["w_out"], w["b_out"], w["labels"])
    G_ref, g0_ref = orn.backward_chain(h32.astype(np.float64), w["w_hh"], seed)
    dh, dw, dseed = to_gpu(h32), to_gpu(w["w_hh"]), to_gpu(np.asarray(seed, np.float32))
    g0a = torch.empty((B, H), dtype=torch.float32, device="cuda") if want_g0 else None
    g0b = torch.empty((B, H), dtype=torch.float32, device="cuda") if want_g0 else None
    Jt = bp.build_jacobians(bp.RNN_TANH, dh, w_hh=dw)
    G_two = to_np(bp.scan(Jt, dseed, g0=g0a))
    G_fused = to_np(bp.rnn_scan_fused(dh, dw, dseed, g0=g0b))
    torch.cuda.synchronize()
    assert np.array_equal(G_fused, G_two)
    assert rel_err(G_fused, G_ref) <= TOL
    if want_g0:
        assert np.array_equal(to_np(g0a), to_np(g0b))
        assert rel_err(to_np(g0b), g0_ref) <= TOL * max(1.0, np.max(np.abs(G_ref)) / max(np.max(np.abs(g0_ref)), 1e-300))


@pytest.mark.parametrize("T,B", [(3000, 5), (3001, 4), (3300, 7), (1000, 13), (1001, 13), (1500, 23), (1100, 14), (1001, 9)])
def test_scan_h20_chains_on_dies_of_unequal_shares(bp, T, B):
    """Batches of four to seven and of thirteen to twenty-three samples keep each chain on one die; either side of the
    lengths from which they do, stored and generated matrices."""
    w = workloads.rnn_inputs_norm_preserving(T, B, seed=T + B, gain=1.05)
    h = np.asarray(orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"]), np.float32)
    seed = np.random.default_rng(B).standard_normal((B, 20)).astype(np.float32)
    G_ref, _ = orn.backward_chain(h.astype(np.float64), w["w_hh"], seed.astype(np.float64))
    dh, dw, dseed = to_gpu(h), to_gpu(w["w_hh"]), to_gpu(seed)
    stored = to_np(bp.scan(bp.build_jacobians(bp.RNN_TANH, dh, w_hh=dw), dseed))
    generated = to_np(bp.rnn_scan_fused(dh, dw, dseed))
    assert np.array_equal(stored, generated)
    assert rel_err(stored, G_ref) <= TOL


@pytest.mark.parametrize("T,B,want_g0", [(1, 3, True), (2, 1, False), (16, 2, True), (17, 5, False), (18, 3, False), (32, 1, True),
                                         (33, 40, False), (49, 7, True), (100, 16, False), (300, 256, False), (70, 300, True)])
def test_h20_scan_as_a_serial_chain(bp, T, B, want_g0):
    """Sizes the scan walks as one chain per sample (short ones, wide ones), around its chunks of 16; both sources of
    the Jacobians and the products of the tree agree with the oracle, and the error word is cleared."""
    import torch
    rng = np.random.default_rng(T + B)
    w_hh = (rng.uniform(-1, 1, (20, 20)) / np.sqrt(20)).astype(np.float32)
    h = np.tanh(rng.standard_normal((T + 1, B, 20))).astype(np.float32)
    seed = rng.standard_normal((B, 20)).astype(np.float32)
    dh, dw, dseed = to_gpu(h), to_gpu(w_hh), to_gpu(seed)
    g0 = [torch.full((B, 20), np.nan, device="cuda") if want_g0 else None for _ in range(2)]
    Jt = bp.build_jacobians(bp.RNN_TANH, dh, w_hh=dw)
    ws = _ws(bp, T, B)
    out = [to_np(bp.scan(Jt, dseed, g0=g0[0], workspace=ws)), to_np(bp.rnn_scan_fused(dh, dw, dseed, g0=g0[1]))]
    assert _error_word(ws) == 0
    ref, g0_ref = oscan.linear_scan(orn.jacobians_T(h, w_hh), seed)
    assert np.array_equal(out[0], out[1]) and rel_err(out[0], ref) <= TOL
    if want_g0:
        assert np.array_equal(to_np(g0[0]), to_np(g0[1]))
        assert rel_err(to_np(g0[0]), g0_ref) <= TOL


def test_rnn_scan_fused_rejects_other_sizes(bp):
    import torch
    h = torch.zeros((5, 2, 16), dtype=torch.float32, device="cuda")
    w = torch.zeros((16, 16), dtype=torch.float32, device="cuda")
    s = torch.zeros((2, 16), dtype=torch.float32, device="cuda")
    with pytest.raises(bp.BppsaError):
        bp.rnn_scan_fused(h, w, s)


def test_three_calls_can_be_captured_in_a_hip_graph(bp):
    """The hot-path calls enqueue kernels only (no allocation, no memset node), so a caller may
    capture them; every replay, with eager work in between, must reproduce the eager result."""
    import torch
    w = workloads.rnn_inputs(200, 16, 20, 1, 10, seed=5)
    T, B, H, I = 200, 16, 20, 1
    d = {k: to_gpu(w[k]) for k in ("x", "w_ih", "w_hh", "b", "w_out", "b_out")}
    h = torch.zeros((T + 1, B, H), dtype=torch.float32, device="cuda")
    bp.forward(bp.RNN_TANH, d["x"], d["w_ih"], d["w_hh"], d["b"], None, h)
    seed, _ = bp.head_seed(h[-1].contiguous(), d["w_out"], d["b_out"], to_gpu(w["labels"]))
    Jt = torch.empty((T, B, H, H), dtype=torch.float32, device="cuda")
    G = torch.empty((T, B, H), dtype=torch.float32, device="cuda")
    ws = torch.empty(bp.scan_workspace_bytes(T, B, H), dtype=torch.uint8, device="cuda")
    pws = torch.empty(max(bp.param_grads_workspace_bytes(bp.RNN_TANH, T, B, H, I), 256), dtype=torch.uint8, device="cuda")
    out = (torch.empty((H, I), device="cuda"), torch.empty((H, H), device="cuda"),
           torch.empty((H,), device="cuda"), torch.empty((H,), device="cuda"))

    def step():
        bp.build_jacobians(bp.RNN_TANH, h, w_hh=d["w_hh"], Jt=Jt)
        bp.scan(Jt, seed, G=G, g0=None, workspace=ws)
        bp.param_grads(bp.RNN_TANH, h, d["x"], G, out=out, workspace=pws)

    step()
    torch.cuda.synchronize()
    ref = [t.clone() for t in out] + [G.clone()]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(4):
        G.zero_()
        for t in out:
            t.zero_()
        ws.fill_(0xAB)                         # the workspace may hold anything between calls
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, r) for a, r in zip(list(out) + [G], ref))
        step()                                  # eager work between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("T,B", [(1, 8), (1, 3), (40, 16), (70, 5)])
def test_scan_h20_error_word_is_zero_after_a_normal_call(bp, T, B):
    """The workspace may hold anything on entry; its first word reads 0 after a normal call."""
    import torch
    jt, seed = workloads.random_jacobian_chain(T, B, 20, seed=T + B)
    ws = torch.full((bp.scan_workspace_bytes(T, B, 20),), 0xC3, dtype=torch.uint8, device="cuda")
    G = bp.scan(to_gpu(jt), to_gpu(seed), workspace=ws)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    assert np.array_equal(to_np(G[T - 1]), seed)
