"""GPU: bppsa_forward where it walks a long sequence as segments at the same time.  Whatever the weights, the states
are those of the walk from the start: compared with the same call on pieces too short to be cut, and with the oracle."""
import numpy as np
import pytest

import workloads
from oracle import gru as ogru
from oracle import rnn as orn
from util import to_gpu, to_np

pytestmark = pytest.mark.gpu

PIECE = 96           # no sequence below 120 steps is cut; even, as the wave form alternates between even and odd steps


@pytest.fixture(scope="module")
def bp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1907_10134_amd as lib
    return lib


def _inputs(cell, T, B, H, I, gain, seed=0):
    rng = np.random.default_rng(seed + T + H)
    w = workloads.rnn_inputs(T, B, H, I, 10, seed=T + H) if cell == "rnn" else workloads.gru_inputs(T, B, H, I, 11, seed=T + H)
    if cell == "rnn":
        w["b_ih"], w["b_hh"] = w["b"], None
    w["w_hh"] = (gain * w["w_hh"]).astype(np.float32)
    return w, (0.3 * rng.standard_normal((B, H))).astype(np.float32)


def _run(bp, cell, w, h0, piece=None):
    import torch
    T, B, _ = w["x"].shape
    h = torch.full((T + 1,) + h0.shape, 7.0, dtype=torch.float32, device="cuda")
    h[0] = to_gpu(h0)
    x = to_gpu(w["x"])
    weights = [None if w[k] is None else to_gpu(w[k]) for k in ("w_ih", "w_hh", "b_ih", "b_hh")]
    code = bp.RNN_TANH if cell == "rnn" else bp.GRU
    step = piece or T
    for t in range(0, T, step):
        n = min(step, T - t)
        bp.forward(code, x[t:t + n], *weights, h[t:t + n + 1])
    return to_np(h)


def _oracle(cell, w, h0):
    if cell == "rnn":
        return orn.forward(w["x"], w["w_ih"], w["w_hh"], w["b"], h0=h0)
    ref = [h0.astype(np.float64)]
    for x in w["x"]:
        ref.append(ogru.step(ref[-1], x, w["w_ih"], w["w_hh"], w["b_ih"], w["b_hh"]))
    return np.asarray(ref)


SIZES = [("rnn", 1000, 16, 20, 1), ("rnn", 337, 3, 20, 1), ("rnn", 1009, 5, 20, 4), ("rnn", 513, 2, 5, 1), ("rnn", 600, 3, 8, 3),
         ("rnn", 301, 7, 9, 1), ("rnn", 272, 1, 21, 1), ("rnn", 499, 2, 32, 2), ("rnn", 999, 700, 20, 1), ("rnn", 300, 7, 64, 1),
         ("rnn", 351, 2, 33, 5), ("rnn", 288, 1, 128, 40), ("rnn", 400, 2, 20, 5), ("gru", 517, 4, 20, 24), ("gru", 333, 3, 8, 12),
         ("gru", 260, 2, 33, 2), ("gru", 700, 1, 97, 33), ("gru", 250, 5, 128, 1), ("gru", 300, 1, 64, 13)]


@pytest.mark.parametrize("cell,T,B,H,I", SIZES)
def test_segments_match_the_oracle(bp, cell, T, B, H, I):
    w, h0 = _inputs(cell, T, B, H, I, 1.0)
    got, ref = _run(bp, cell, w, h0), _oracle(cell, w, h0)
    assert np.max(np.abs(got - ref)) <= 2e-6          # as for sequences walked in one go
    assert np.max(np.abs(got - _run(bp, cell, w, h0, PIECE))) <= 2e-6


@pytest.mark.parametrize("cell,T,B,H,I", [s for s in SIZES if s[2] < 100])
def test_segments_of_cells_that_amplify(bp, cell, T, B, H, I):
    """Chaotic weights: a wrong start would show at the size of the states, which are O(1), at the next seam at the
    latest.  Seams that do not hold are walked again, so what is left is the walk from the start."""
    w, h0 = _inputs(cell, T, B, H, I, 12.0)
    assert np.max(np.abs(_run(bp, cell, w, h0) - _run(bp, cell, w, h0, PIECE))) <= 2e-6


@pytest.mark.parametrize("gain", [2.0, 3.0])
@pytest.mark.parametrize("cell,T,B,H,I", [s for s in SIZES if s[2] < 100])
def test_segments_of_cells_that_forget_slowly(bp, cell, T, B, H, I, gain):
    """Some seams hold, some do not, and what a seam leaves (2^-20 of the largest state) may grow as the rounding of
    every step does: the states are about as far from the oracle's as those of the walk from the start."""
    w, h0 = _inputs(cell, T, B, H, I, gain)
    ref = _oracle(cell, w, h0)
    off, base = (np.linalg.norm(_run(bp, cell, w, h0, p) - ref) for p in (None, PIECE))
    assert off <= 2 * base + 1e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("T,B", [(700, 3), (1500, 16)])
def test_segments_with_a_norm_preserving_recurrence(bp, T, B):
    """No seam holds: the bits of the walk from the start."""
    w = workloads.rnn_inputs_norm_preserving(T, B, seed=T)
    w["b_ih"], w["b_hh"] = w["b"], None
    h0 = np.zeros((B, 20), np.float32)
    assert np.array_equal(_run(bp, "rnn", w, h0), _run(bp, "rnn", w, h0, PIECE))


@pytest.mark.parametrize("cell,T,B,H,I", [("rnn", 600, 4, 20, 1), ("rnn", 400, 4, 64, 1), ("gru", 517, 4, 20, 24)])
def test_a_nan_in_one_sample_goes_on_to_its_end_and_nowhere_else(bp, cell, T, B, H, I):
    w, h0 = _inputs(cell, T, B, H, I, 1.0)
    clean = _run(bp, cell, w, h0)
    w["x"] = w["x"].copy()
    w["x"][T // 3, 1, 0] = np.nan
    got = _run(bp, cell, w, h0)
    assert np.isnan(got[T // 3 + 1:, 1]).all()
    assert np.array_equal(got[:T // 3 + 1, 1], clean[:T // 3 + 1, 1])
    assert np.array_equal(np.delete(got, 1, axis=1), np.delete(clean, 1, axis=1))


@pytest.mark.parametrize("gain", [1.0, 12.0])
@pytest.mark.parametrize("T,B,H,I", [(700, 5, 20, 1), (333, 3, 8, 2), (1000, 2, 31, 4)])
def test_training_iteration_on_segments_takes_the_last_state(bp, T, B, H, I, gain):
    """The head of an iteration runs behind the seams: its seed is that of the states as they end up."""
    import torch
    rng = np.random.default_rng(T)
    shapes = bp.binding.rnn_param_shapes(H, I, 10)
    p = {k: torch.from_numpy((rng.uniform(-1, 1, shapes[k]) / np.sqrt(H)).astype(np.float32)).cuda() for k in bp.RNN_PARAM_ORDER}
    p["w_hh"] *= gain
    x = to_gpu(rng.standard_normal((T, B, I)).astype(np.float32))
    labels = to_gpu(rng.integers(0, 10, B).astype(np.int32))
    tr = bp.RnnTrainer(T, B, H, I, 10, {k: v.clone() for k, v in p.items()})
    tr.step(x, labels)
    h = torch.zeros_like(tr.h)
    bp.forward(bp.RNN_TANH, x, p["w_ih"], p["w_hh"], p["b_ih"], p["b_hh"], h)
    assert torch.equal(h, tr.h)
    seed, _ = bp.head_seed(h[T], p["w_out"], p["b_out"], labels)
    assert torch.allclose(tr.seed, seed, rtol=1e-5, atol=1e-8)


# more samples than segments have room for, up to the compute units, and one more than those
ROUNDS = [(288, 100, 20, 1), (289, 65, 20, 1), (290, 256, 5, 2), (385, 130, 8, 4), (1000, 100, 32, 1), (611, 256, 9, 3),
          (400, 257, 20, 1)]


@pytest.mark.parametrize("gain", [1.0, 2.0, 12.0])
@pytest.mark.parametrize("T,B,H,I", ROUNDS)
def test_rounds_of_walks(bp, T, B, H, I, gain):
    w, h0 = _inputs("rnn", T, B, H, I, gain)
    got, pieces = _run(bp, "rnn", w, h0), _run(bp, "rnn", w, h0, PIECE)
    if gain == 2.0:                                   # as above for cells that forget slowly
        ref = _oracle("rnn", w, h0)
        assert np.linalg.norm(got - ref) <= 2 * np.linalg.norm(pieces - ref) + 1e-7 * np.linalg.norm(ref)
    else:
        assert np.max(np.abs(got - pieces)) <= 2e-6
