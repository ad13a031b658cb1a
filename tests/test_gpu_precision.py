"""fp32 contractions on the bf16 matrix cores keep the precision of the fp32 ones: errors against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1502_00512_amd import binding, synth
from test_gpu_parity import dev

pytestmark = pytest.mark.gpu

FP32 = binding.RNNLM_FP32


def distance(got, ref):
    return np.linalg.norm(got.detach().cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)


def gradients(E, U, Wo, b, x, y):
    T, B = x.shape
    g = binding.Rnnlm(E, U, Wo, b, B, T, FP32)
    r = g.rnnlm_grad_chunk(dev(x), dev(y))
    g.rnnlm_check()
    g.close()
    return r


# each tile form of the fp32 contractions at least once
@pytest.mark.parametrize("V,H,B,T", [
    (600, 200, 64, 30), (900, 900, 5, 40), (2000, 300, 60, 20), (10000, 256, 32, 10), (30000, 100, 128, 8), (20000, 300, 128, 16),
    (20000, 500, 64, 8), (5000, 1500, 20, 20),
])
def test_no_product_of_the_split_operands_is_lost(V, H, B, T):
    """The bounds lie between what is right and what a lost product leaves.  Gradients: measured 0.7e-7 to 2.9e-7; an operand
    of 16 bits (no products of its lowest part) 2.3e-6 to 2.8e-6.  Log-probabilities, with weights of up to 1, which spread the
    logits: a logit is rounded 6 H / 16 times where one accumulator takes all products (sqrt(190) 2^-25 = 4e-7 of it at H =
    500; measured 2.7e-7 at most); 16-bit weights 4.2e-7 to 9.1e-7."""
    scale = 0.1 if H < 512 else 0.05
    E, U, Wo, b = synth.make_weights(V, H, "uniform", scale, V)
    tok = synth.zipf_tokens(B * T + B + 1, V, 1.05, 3)
    x, y = O.stream_chunk(tok, B, T, 0)
    r, ref = gradients(E, U, Wo, b, x, y), O.grad_chunk(O.Model.from_weights(E, U, Wo, b, B), x, y)
    for k in ("gE", "gU", "gWo"):
        assert distance(r[k], ref[k]) <= 8e-7, (k, distance(r[k], ref[k]))
    Wo = Wo * np.float32(1 / scale)
    g = binding.Rnnlm(E, U, Wo, b, B, T, FP32)
    got, want = g.rnnlm_forward_logprob(dev(x), dev(y)), O.forward_logprob(O.Model.from_weights(E, U, Wo, b, B), x, y)
    assert distance(got, want) <= 3.6e-7, distance(got, want)
    g.close()


@pytest.mark.parametrize("V,H,B,T", [
    (400, 1000, 256, 40), (1600, 1000, 512, 30), (3209, 852, 512, 32), (1200, 700, 100, 20), (20000, 300, 128, 16),
])
def test_gradients_through_the_vocabulary_are_as_close_as_the_fp32_cores_bring_them(V, H, B, T):
    """An operand that a bf16 cannot hold makes a tile fall back to the fp32 matrix cores.  Here every 32nd word never
    occurs and has probability 0, once because of its bias and once because it has such a weight in every block of 64
    columns: the same gradients, formed on the bf16 cores and on the fp32 ones."""
    E, U, Wo, b = synth.make_weights(V, H, "uniform", 0.1 if H < 512 else 0.05, V)
    dead = np.arange(7, V, 32)
    tok = synth.zipf_tokens(B * T + B + 1, V, 1.05, 3)
    tok = np.where(np.isin(tok, dead), tok - 1, tok).astype(np.int32)
    x, y = O.stream_chunk(tok, B, T, 0)
    b[dead] = -1e30
    ref = O.grad_chunk(O.Model.from_weights(E, U, Wo, b, B), x, y)
    split = gradients(E, U, Wo, b, x, y)
    Wo[np.ix_(dead, np.arange(5, H, 64))] = -3.4e38
    cores = gradients(E, U, Wo, b, x, y)
    assert not torch.equal(split["gU"], cores["gU"])
    # (in the recurrent gradient its own contraction, the same on both sides, adds rounding of its own: within a few percent
    # where that is most of it)
    for k, room in (("gE", 1.0), ("gU", 1.05)):
        near, far = distance(split[k], ref[k]), distance(cores[k], ref[k])
        assert near <= room * far, (k, near, far)
    assert distance(split["logp"], ref["logp"]) <= 1.1 * distance(cores["logp"], ref["logp"])
