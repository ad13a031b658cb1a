"""The row updates' run sums against the fp64 oracle, at the run lengths where their shape changes: one member, one wave's
share (16) and one more, a slice's 64 positions and one more per wave, a single run of everything; fp32."""
import numpy as np
import pytest
import torch

from oracle import compressed as Cq
from oracle import oracle as O
from paper_1502_00512_amd import binding, synth

pytestmark = pytest.mark.gpu


def tokens_of(lengths, M, V, seed):
    ids = np.random.default_rng(seed).permutation(V)
    flat = np.repeat(ids[:len(lengths)], np.asarray(lengths, int))
    assert len(flat) <= M
    flat = np.concatenate([flat, ids[len(lengths):len(lengths) + M - len(flat)]])  # the rest: runs of one
    return np.random.default_rng(seed + 1).permutation(flat).astype(np.int32)


# H: columns in one, two, five and nine blocks of 256, whole and ragged groups of four
@pytest.mark.parametrize("H", [64, 255, 260, 1024, 2306])
@pytest.mark.parametrize("B,T,lengths", [
    (8, 5, [8, 9, 16]), (8, 5, [17]), (30, 30, [15, 16, 17, 64, 65, 128, 513]), (40, 26, [16, 17, 33, 519, 128]),
    (40, 40, [1600]),
])
def test_embedding_update_by_run_length(H, B, T, lengths):
    V, M, lr = 1700, B * T, 0.5
    E, U, Wo, b = synth.make_weights(V, H, "uniform", 0.1, 3 + H)
    x = tokens_of(lengths, M, V, 11 + H).reshape(T, B)
    y = tokens_of(lengths, M, V, 12 + H).reshape(T, B)
    o = O.Model.from_weights(E, U, Wo, b, B)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    # windows of up to 1024 positions (the first three shapes) compare ids, the rmsprop call sorts them: the same sums, bit
    # for bit (every denominator is exactly one there).  The longer ones are sorted in both calls; what compares ids up to
    # 4096 positions is the compressed architecture below.
    g = binding.Rnnlm(E, U, Wo, b, B, T, binding.RNNLM_FP32)
    s = binding.Rnnlm(E, U, Wo, b, B, T, binding.RNNLM_FP32, rmsprop=True, r_init=1.0)
    g.rnnlm_train_chunk(d(x), d(y), lr)
    s.rnnlm_train_chunk_rmsprop(d(x), d(y), lr, 1.0, 0.0)
    assert torch.equal(g.E, s.E)
    O.train_chunk(o, x, y, lr)
    # the fp32 gradients' bound of the suite (1e-3 of the largest entry) on the step that was taken
    step, ref = g.E.cpu().numpy().astype(np.float64) - E, o.E - E
    assert np.abs(step - ref).max() <= 1e-3 * np.abs(ref).max() + 1.2e-7 * np.abs(E).max()
    assert np.array_equal(g.E.cpu().numpy()[ref.any(1) == 0], E[ref.any(1) == 0])


@pytest.mark.parametrize("H", [64, 255, 1024, 1102])
@pytest.mark.parametrize("noise,targets", [([1] * 7, [16]), ([8, 8], [9]), ([16], [17]), ([300], [513, 130]), ([64], [65, 64])])
def test_noise_contrastive_row_update_by_run_length(H, noise, targets):
    V, B, T = 1200, 30, 25
    K = sum(noise)
    E, U, Wo, b = synth.make_weights(V, H, "uniform", 0.1, 5 + H)
    x = tokens_of([], B * T, V, 21).reshape(T, B)
    y = tokens_of(targets, B * T, V, 22).reshape(T, B)
    nw = tokens_of(noise, K, V, 22)  # the same permutation of the words: noise and target runs meet in one list
    lnq = np.full(V, -np.log(V), np.float32)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    g = binding.Rnnlm(E, U, Wo, b, B, T, binding.RNNLM_FP32, K_max=K)
    o = O.Model.from_weights(E, U, Wo, b, B)
    g.rnnlm_nce_train_chunk(d(x), d(y), d(nw), d(lnq), 2.0, 0.5)
    O.nce_train_chunk(o, x, y, nw, lnq, 2.0, 0.5)
    for got, ref, start in ((g.Wo, o.Wo, Wo), (g.b, o.b, b)):
        step, want = got.cpu().numpy().astype(np.float64) - start, ref - start
        assert np.abs(step - want).max() <= 1e-3 * np.abs(want).max() + 1.2e-7 * np.abs(start).max()


# P: columns in one, two, three and nine blocks of 256, whole and ragged groups of four; the last window is sorted
@pytest.mark.parametrize("precision", [binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER])
@pytest.mark.parametrize("P", [64, 130, 260, 515, 2100])
@pytest.mark.parametrize("B,T,lengths", [
    (32, 33, [16, 17, 33, 519, 128]), (64, 64, [4096]), (64, 64, [15, 16, 17, 64, 65, 128, 129, 513, 1500]), (63, 65, [2100, 8, 9]),
    (64, 65, [16, 17, 513, 64, 65, 1200]),
])
def test_tied_matrix_update_by_run_length(B, T, lengths, P, precision):
    V, H, M, fp32 = 4600, 48, B * T, precision == binding.RNNLM_FP32
    E, A, U, C_, b = synth.make_compressed_weights(V, H, P, "uniform", 0.2, 3 + P)
    x = tokens_of(lengths, M, V, 11 + P).reshape(T, B)
    y = np.full((T, B), V - 1, np.int32)  # (one target: the output-side share of a row is a sum of one sign)
    g = binding.Rnnlm(E, U, None, b, B, T, precision, A=A, C_=C_)
    o = Cq.CompressedModel(*(np.asarray(a, np.float64).copy() for a in (E, A, U, C_, b)), np.zeros((B, H)))
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    ref = Cq.grad_chunk(o, x, y)["gE"]
    got = g.rnnlm_grad_chunk_compressed(d(x), d(y))["gE"].cpu().numpy().astype(np.float64)
    # row by row, fp32: a member too few among 4096 is 2.4e-4 of a row, measured 4.4e-6 at most; bf16: operands of the layers
    # on the way are rounded to 2^-9, P = 2100 measured 3.1e-2 at most
    off, size = np.linalg.norm(got - ref, axis=1), np.linalg.norm(ref, axis=1)
    assert (off <= 2e-5 * size if fp32 else off <= 5e-2 * size).all(), (off / size).max()
    g.rnnlm_train_chunk(d(x), d(y), 0.5)
    g.rnnlm_check()
    # the workspace begins with the compute copy of the tied matrix, rows padded to 256 columns
    Pp, es, dt = -(-P // 256) * 256, 4 if fp32 else 2, torch.float32 if fp32 else torch.bfloat16
    copy = g.workspace[:V * Pp * es].view(dt).view(V, Pp)
    assert torch.equal(copy[:, :P], g.E.to(dt)) and not bool(copy[:, P:].any())
