"""GPU parity: one training iteration of the Section 4.1 RNN (forward, head, backward as a scan,
Adam) through the C ABI against the fp64 oracle on the same seeded bit-stream batches."""
import numpy as np
import pytest

import workloads
from oracle import rnn as orn
from oracle import train as otrain
from util import TOL, rel_err, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1907_10134_amd as lib
    return lib


@pytest.mark.parametrize("T,B,I", [(200, 5, 1), (64, 3, 3), (65, 1, 4), (1, 2, 1), (1000, 16, 1)])
def test_forward_h20_wave_per_sample(bp, T, B, I):
    """The H = 20 forward (one wave per sample) against the oracle's recurrence, every state."""
    import torch
    rng = np.random.default_rng(T + I)
    p = workloads.rnn_parameters(I=I, seed=T)
    x = rng.standard_normal((T, B, I)).astype(np.float32)
    h = torch.zeros((T + 1, B, 20), dtype=torch.float32, device="cuda")
    h0 = (0.1 * rng.standard_normal((B, 20))).astype(np.float32)
    h[0] = to_gpu(h0)
    bp.forward(bp.RNN_TANH, to_gpu(x), to_gpu(p["w_ih"]), to_gpu(p["w_hh"]), to_gpu(p["b_ih"]), to_gpu(p["b_hh"]), h)
    ref = orn.forward(x, p["w_ih"], p["w_hh"], p["b_ih"].astype(np.float64) + p["b_hh"], h0=h0)
    assert np.max(np.abs(to_np(h) - ref)) <= 2e-5        # states are O(1); fp32 tanh and sums


@pytest.mark.parametrize("cell", ["rnn", "gru"])
@pytest.mark.parametrize("T,B,H,I", [(1, 1, 1, 1), (16, 2, 8, 1), (17, 2, 9, 4), (31, 3, 20, 5), (33, 2, 21, 12), (15, 2, 32, 2),
                                     (18, 1, 33, 13), (16, 2, 64, 20), (34, 1, 65, 21), (20, 2, 96, 32), (19, 2, 97, 33),
                                     (40, 1, 128, 40), (9, 1, 128, 41), (7, 1, 129, 1)])
def test_forward_at_the_edges_of_the_recurrence_kernels(bp, cell, T, B, H, I):
    """Hidden sizes, input widths and sequence lengths on both sides of every kernel's limits (units per
    wave, columns per row of lanes, steps per trip, the largest H and I of the register form)."""
    import torch
    from oracle import gru as ogru
    rng = np.random.default_rng(T * 1000 + H)
    h0 = (0.3 * rng.standard_normal((B, H))).astype(np.float32)
    h = torch.zeros((T + 1, B, H), dtype=torch.float32, device="cuda")
    h[0] = to_gpu(h0)
    if cell == "rnn":
        w = workloads.rnn_inputs(T, B, H, I, 10, seed=T + H)
        bp.forward(bp.RNN_TANH, to_gpu(w["x"]), to_gpu(w["w_ih"]), to_gpu(w["w_hh"]), to_gpu(w["b"]), None, h)
        ref = orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"], h0=h0)
    else:
        w = workloads.gru_inputs(T, B, H, I, 11, seed=T + H)
        bp.forward(bp.GRU, *(to_gpu(w[k]) for k in ("x", "w_ih", "w_hh", "b_ih", "b_hh")), h)
        ref = [h0.astype(np.float64)]
        for t in range(T):
            ref.append(ogru.step(ref[t], w["x"][t], w["w_ih"], w["w_hh"], w["b_ih"], w["b_hh"]))
    assert np.max(np.abs(to_np(h) - np.asarray(ref))) <= 2e-6


@pytest.mark.parametrize("B,H,C", [(16, 20, 10), (256, 20, 10), (3, 128, 11), (1, 20, 1), (100, 7, 64)])
def test_head_backward_matches_oracle(bp, B, H, C):
    rng = np.random.default_rng(B + H)
    h_last = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    w_out = (rng.standard_normal((C, H)) / np.sqrt(H)).astype(np.float32)
    b_out = (0.1 * rng.standard_normal(C)).astype(np.float32)
    labels = rng.integers(0, C, B).astype(np.int32)
    seed, loss, dW, db = bp.head_backward(to_gpu(h_last), to_gpu(w_out), to_gpu(b_out), to_gpu(labels))
    l_ref, s_ref, dW_ref, db_ref = otrain.head_backward(h_last, w_out, b_out, labels)
    assert abs(float(to_np(loss)[0]) - l_ref) <= 1e-5 * max(1.0, abs(l_ref))
    assert rel_err(to_np(seed), s_ref) <= TOL
    assert rel_err(to_np(dW), dW_ref) <= TOL
    assert np.max(np.abs(to_np(db) - db_ref)) <= 1e-6
    # the older entry point gives the same seed and loss
    seed2, loss2 = bp.head_seed(to_gpu(h_last), to_gpu(w_out), to_gpu(b_out), to_gpu(labels))
    assert rel_err(to_np(seed2), s_ref) <= TOL and abs(float(to_np(loss2)[0]) - l_ref) <= 1e-5 * max(1.0, abs(l_ref))


@pytest.mark.parametrize("B,H,C", [(15, 19, 16), (17, 3, 17), (33, 31, 33), (300, 64, 2), (64, 128, 11), (1000, 4, 10),
                                   (40, 900, 3), (2, 5000, 5), (5, 129, 64)])
def test_head_backward_at_the_edges_of_its_tiles(bp, B, H, C):
    """Batches, widths and classes around the tiles of 16, and heads that do not fit into LDS."""
    rng = np.random.default_rng(B + H)
    h_last = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    w_out = (rng.standard_normal((C, H)) / np.sqrt(H)).astype(np.float32)
    b_out = (0.1 * rng.standard_normal(C)).astype(np.float32)
    labels = rng.integers(0, C, B).astype(np.int32)
    out = bp.head_backward(to_gpu(h_last), to_gpu(w_out), to_gpu(b_out), to_gpu(labels))
    l_ref, s_ref, dW_ref, db_ref = otrain.head_backward(h_last, w_out, b_out, labels)
    for got, ref in zip(out, (s_ref, [l_ref], dW_ref, db_ref)):
        assert rel_err(to_np(got), np.asarray(ref)) <= TOL


@pytest.mark.parametrize("T,B,H,I,C", [(9, 3, 8, 1, 10), (16, 2, 20, 4, 64), (17, 40, 20, 2, 3), (31, 5, 31, 3, 11),
                                       (33, 2, 32, 4, 10), (12, 3, 33, 1, 10), (10, 2, 20, 5, 10)])
def test_training_iteration_at_the_edges_of_the_fused_launches(bp, T, B, H, I, C):
    """Sizes with the head in the forward launch (H <= 32, at most four inputs) and without; the parts called one by
    one give the gradients and the updated parameters."""
    import torch
    rng = np.random.default_rng(T * B + H)
    shapes = bp.binding.rnn_param_shapes(H, I, C)
    params = {k: (rng.uniform(-1, 1, shapes[k]) / np.sqrt(H)).astype(np.float32) for k in bp.RNN_PARAM_ORDER}
    x = rng.standard_normal((T, B, I)).astype(np.float32)
    labels = rng.integers(0, C, B).astype(np.int32)
    tr = bp.RnnTrainer(T, B, H, I, C, {k: torch.from_numpy(v) for k, v in params.items()})
    loss = tr.step(to_gpu(x), to_gpu(labels), lr=1e-3)
    p64 = {k: v.astype(np.float64) for k, v in params.items()}
    l_ref, g_ref, p_ref, _ = otrain.rnn_iteration(p64, otrain.zero_moments(p64), x, labels, 1, lr=1e-3)
    assert abs(float(to_np(loss)[0]) - l_ref) <= 1e-5 * max(1.0, abs(l_ref))
    for k in g_ref:
        assert rel_err(to_np(tr.view(tr.grads, k)), g_ref[k]) <= 5 * TOL, k
        assert np.max(np.abs(to_np(tr.view(tr.params, k)) - p_ref[k])) <= 2e-5, k


@pytest.mark.parametrize("T,B,I,C", [(2, 1, 1, 10), (3, 5, 2, 1), (10, 180, 3, 64), (100, 7, 4, 17), (288, 80, 1, 10),
                                     (289, 80, 2, 16), (500, 256, 1, 10), (400, 257, 4, 10)])
def test_training_iteration_walked_both_ways_in_one_launch(bp, T, B, I, C):
    """H = 20 with generated Jacobians: sequences of one walk and of rounds, more samples than compute units, classes
    that the standard workspace has room for and that it has not; and the same on the least workspace that is taken."""
    import torch
    rng = np.random.default_rng(T * B + I)
    shapes = bp.binding.rnn_param_shapes(20, I, C)
    params = {k: (rng.uniform(-1, 1, shapes[k]) / np.sqrt(20)).astype(np.float32) for k in bp.RNN_PARAM_ORDER}
    x = rng.standard_normal((T, B, I)).astype(np.float32)
    labels = rng.integers(0, C, B).astype(np.int32)
    p64 = {k: v.astype(np.float64) for k, v in params.items()}
    l_ref, g_ref, p_ref, _ = otrain.rnn_iteration(p64, otrain.zero_moments(p64), x, labels, 1, lr=1e-3)

    def check(tr):
        tr.G.fill_(7.0)
        loss = tr.step(to_gpu(x), to_gpu(labels), lr=1e-3)
        assert abs(float(to_np(loss)[0]) - l_ref) <= 1e-5 * max(1.0, abs(l_ref))
        for k in g_ref:
            assert rel_err(to_np(tr.view(tr.grads, k)), g_ref[k]) <= TOL, k
            assert np.max(np.abs(to_np(tr.view(tr.params, k)) - p_ref[k])) <= 2e-5, k
        h = torch.zeros_like(tr.h)
        w = [to_gpu(params[k]) for k in ("w_ih", "w_hh", "b_ih", "b_hh")]
        bp.forward(bp.RNN_TANH, to_gpu(x), *w, h)
        G = bp.rnn_scan_fused(h, w[1], tr.seed)
        assert np.max(np.abs(to_np(tr.h) - to_np(h))) <= 2e-6
        assert rel_err(to_np(tr.G), to_np(G)) <= TOL

    def trainer():
        return bp.RnnTrainer(T, B, 20, I, C, {k: torch.from_numpy(v) for k, v in params.items()}, materialise=False)

    check(trainer())
    probe, lo, hi = trainer(), 0, trainer().workspace.numel()
    while hi - lo > 1:
        probe._st.workspace_bytes = (lo + hi) // 2
        try:
            probe.step(to_gpu(x), to_gpu(labels))
            hi = (lo + hi) // 2
        except bp.BppsaError:
            lo = (lo + hi) // 2
    least = trainer()
    least._st.workspace_bytes = hi
    check(least)


def test_adam_step_matches_oracle_over_several_steps(bp):
    rng = np.random.default_rng(3)
    n = 1000
    theta = rng.standard_normal(n).astype(np.float32)
    th_ref, m_ref, v_ref = theta.astype(np.float64), np.zeros(n), np.zeros(n)
    th, m, v = to_gpu(theta), to_gpu(np.zeros(n, np.float32)), to_gpu(np.zeros(n, np.float32))
    for t in range(1, 8):
        g = (rng.standard_normal(n) * 10.0 ** rng.integers(-6, 1, n)).astype(np.float32)
        g[:10] = 0.0
        bp.adam_step(th, to_gpu(g), m, v, t, lr=1e-3)
        th_ref, m_ref, v_ref = otrain.adam_step(th_ref, g, m_ref, v_ref, t, lr=1e-3)
    # seven steps of at most lr each; every step is accurate to fp32 rounding of a ratio of O(1)
    assert np.max(np.abs(to_np(th) - th_ref)) <= 7 * 1e-3 * 1e-5 + 1e-6
    assert rel_err(to_np(m), m_ref) <= 1e-5 and rel_err(to_np(v), v_ref) <= 1e-5
    assert np.array_equal(to_np(th)[:10], theta[:10])          # zero gradient: untouched


def _run_iterations(bp, T, B, iters, materialise, lr):
    import torch
    params = workloads.rnn_parameters()
    tr = bp.RnnTrainer(T, B, 20, 1, 10, {k: torch.from_numpy(v) for k, v in params.items()}, materialise=materialise)
    p_ref = {k: v.astype(np.float64) for k, v in params.items()}
    mom = otrain.zero_moments(p_ref)
    out = []
    for it in range(iters):
        x, labels = workloads.bitstream_batch(T, B, first_sample=it * B)
        loss = tr.step(to_gpu(x), to_gpu(labels), lr=lr)
        bp.check_scan(tr.workspace)          # synchronises; the scan's error word is still there
        l_ref, g_ref, p_ref, mom = otrain.rnn_iteration(p_ref, mom, x, labels, it + 1, lr=lr)
        out.append((float(to_np(loss)[0]), l_ref, {k: to_np(tr.view(tr.grads, k)).copy() for k in bp.RNN_PARAM_ORDER},
                    g_ref, {k: to_np(tr.view(tr.params, k)).copy() for k in bp.RNN_PARAM_ORDER}, dict(p_ref)))
    return out


@pytest.mark.parametrize("T,B,materialise", [(60, 4, True), (60, 4, False), (1000, 16, False), (1000, 16, True),
                                             (333, 7, False)])
def test_training_iterations_match_oracle(bp, T, B, materialise):
    """Several iterations on fresh batches: the loss, every parameter gradient and the parameters
    after each Adam update against the oracle's iteration.  The oracle carries its own fp64
    parameters forward, so differences accumulate; with lr = 1e-3 each update moves an entry by at
    most lr, and the two sides' updates differ by the relative error of the gradient."""
    iters, lr = 4, 1e-3
    for it, (loss, l_ref, g, g_ref, p, p_ref) in enumerate(_run_iterations(bp, T, B, iters, materialise, lr)):
        assert abs(loss - l_ref) <= 1e-5 * max(1.0, abs(l_ref)) * (it + 1), (it, loss, l_ref)
        for k in g:
            assert rel_err(g[k], g_ref[k]) <= 5 * TOL, (it, k)
            assert np.max(np.abs(p[k] - p_ref[k])) <= (it + 1) * lr * 2e-2, (it, k)


def test_training_with_the_paper_learning_rate_moves_every_parameter(bp):
    """lr = 1e-5 (Section 4.1): after one update every parameter has moved by about lr against the
    sign of its gradient, as the first Adam step does."""
    (loss, l_ref, g, g_ref, p, p_ref), = _run_iterations(bp, 100, 8, 1, False, 1e-5)
    p0 = workloads.rnn_parameters()
    for k in g:
        big = np.abs(g_ref[k]) > 1e-6
        moved = p[k] - p0[k]
        assert np.all(np.sign(moved[big]) == -np.sign(g_ref[k][big]))
        assert np.allclose(np.abs(moved[big]), 1e-5, rtol=0.05, atol=3e-8)     # fp32 spacing near 0.2 is 1.5e-8
