"""GPU parity of the persistent recurrent kernel over the forms its launch rule picks (number of 32-wide contraction
blocks per wave, one or two 16-row blocks of streams, four or eight waves, streams per group): fp32 against the fp64 CPU
oracle at test_gpu_parity.py's tolerances; bf16 bitwise between the two state exchanges and between a window scored
with all its streams and with a few of them (the order of every sum depends on the hidden size alone)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1502_00512_amd import binding, synth
from test_gpu_parity import check_grad, check_logp, dev, make_pair, tokens

pytestmark = pytest.mark.gpu

FP32, BF16 = binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER


@pytest.mark.parametrize("V,H,B,T", [
    (300, 8, 1, 3),       # one workgroup, one wave with work
    (300, 33, 9, 4),      # two streams per group, the last group one
    (300, 161, 130, 3),   # 17 streams per group: two row blocks
    (300, 290, 17, 2),    # 10 blocks over four waves: the last wave has one
    (300, 1000, 200, 2),  # 25 streams per group, 32 blocks
    (300, 1100, 1, 8),    # one launch pair per step: one stream, the window's rows a multiple of nothing
    (300, 1600, 70, 4),   # the same, two 64-row tiles
])
def test_fp32_against_oracle(V, H, B, T):
    g, o = make_pair(V, H, B, T, FP32, seed=V + H + B, scale=0.3 if H < 100 else 0.05, bias_scale=0.5)
    tok = tokens(V, 2 * B * T + B + 1, 6)
    x, y = O.stream_chunk(tok, B, T, 0)
    g.rnnlm_forward_logprob(dev(x), dev(y))
    O.forward_logprob(o, x, y)
    assert np.abs(g.h_state.cpu().numpy() - o.h).max() < 2e-5
    x, y = O.stream_chunk(tok, B, T, 1)
    r = g.rnnlm_grad_chunk(dev(x), dev(y))
    ref = O.grad_chunk(o, x, y)
    check_logp(r["logp"], ref["logp"])
    for k in ("gE", "gU", "gWo", "gb"):
        check_grad(k, r[k], ref[k])
    g.rnnlm_check()


# steps in one launch of their own: one, two and four blocks of 16 streams a workgroup, the last one partly filled, units
# and pieces of the contraction that are no multiple of a workgroup's; and past them, two launches a step
@pytest.mark.parametrize("H,B,T,precision", [
    (1025, 16, 3, FP32), (1100, 17, 2, FP32), (1500, 33, 2, FP32), (1290, 100, 3, FP32), (1600, 200, 2, FP32),
    (2049, 1, 4, BF16), (2064, 16, 3, BF16), (2300, 31, 2, BF16), (2500, 63, 3, BF16), (2060, 65, 2, BF16), (2500, 130, 2, BF16),
])
def test_wide_layers_step_by_step(H, B, T, precision):
    V = 300
    g, o = make_pair(V, H, B, T, precision, seed=H + B, scale=0.03, bias_scale=0.5)
    tok = tokens(V, 2 * B * T + B + 1, 6)
    x, y = O.stream_chunk(tok, B, T, 0)
    g.rnnlm_forward_logprob(dev(x), dev(y))
    O.forward_logprob(o, x, y)
    # the bounds of the suite: fp32 2e-5 on states; bf16 states, of at most 1, to a few roundings of 2^-9
    assert np.abs(g.h_state.cpu().numpy() - o.h).max() < (2e-5 if precision == FP32 else 2e-2)
    x, y = O.stream_chunk(tok, B, T, 1)
    r = g.rnnlm_grad_chunk(dev(x), dev(y))
    ref = O.grad_chunk(o, x, y)
    for k in ("gE", "gU", "gWo", "gb"):
        a = r[k].cpu().numpy().astype(np.float64)
        assert np.abs(a - ref[k]).max() <= (1e-3 if precision == FP32 else 2e-2) * np.abs(ref[k]).max(), k
    g.rnnlm_check()


@pytest.mark.parametrize("H,B,few", [(40, 256, 3), (200, 100, 1), (650, 250, 7), (1024, 129, 16), (1100, 256, 5), (2000, 120, 9)])
def test_bf16_exchange_and_group_size(H, B, few):
    V, T = 500, 5
    E, U, Wo, b = synth.make_weights(V, H, "normal", 0.1 if H < 500 else 0.03, 3)
    x = tokens(V, T * B, 11).reshape(T, B)
    y = tokens(V, T * B, 12).reshape(T, B)

    def run(n, mode):
        m = binding.Rnnlm(E, U, Wo, b, n, T, BF16)
        try:
            m.rnnlm_set_recurrent_exchange(mode)
        except binding.RnnlmError:
            pytest.skip("this device does not place workgroups round-robin over 8 XCDs: no XCD-local exchange")
        for _ in range(3):
            m.rnnlm_forward_logprob(dev(x[:, :n]), dev(y[:, :n]))
        grads = m.rnnlm_grad_chunk(dev(x[:, :n]), dev(y[:, :n]))
        m.rnnlm_check()
        return m.h_state.cpu(), grads

    h, g = run(B, binding.RNNLM_EXCHANGE_XCD_LOCAL)
    hc, gc = run(B, binding.RNNLM_EXCHANGE_CHIP_WIDE)
    assert torch.equal(h, hc)
    for k in g:
        assert torch.equal(g[k], gc[k]), k
    hf, _ = run(few, binding.RNNLM_EXCHANGE_XCD_LOCAL)
    assert torch.equal(h[:few], hf)


@pytest.mark.parametrize("H,B,T", [(2100, 1, 8), (2400, 64, 4), (4000, 33, 3), (4096, 128, 2)])
def test_bf16_per_step_against_oracle(H, B, T):
    """Hidden sizes beyond the persistent kernel.  Tolerances: the state is rounded to bf16 (2^-9) each step; log-probs
    and gradients as in test_gpu_parity.py's bf16 comparisons."""
    V = 300
    E, U, Wo, b = synth.make_weights(V, H, "normal", 0.02, 5)
    g = binding.Rnnlm(E, U, Wo, b, B, T, BF16)
    o = O.Model.from_weights(E, U, Wo, b, B)
    tok = tokens(V, B * T + B + 1, 8)
    x, y = O.stream_chunk(tok, B, T, 0)
    r = g.rnnlm_grad_chunk(dev(x), dev(y))
    ref = O.grad_chunk(o, x, y)
    assert np.abs(r["logp"].cpu().numpy() - ref["logp"]).max() < 2e-2
    for k in ("gE", "gU", "gWo", "gb"):
        d = r[k].cpu().numpy() - ref[k]
        assert np.linalg.norm(d) <= 2e-2 * np.linalg.norm(ref[k]), k
    g.rnnlm_check()


def test_bf16_state_to_state_matrix_of_2_gib():
    """H = 32768: the per-step backward product's K-major operand is beyond the direct-load kernels' offsets.  One window
    against 64-bit arithmetic on the device (the oracle would take minutes); tolerances as above."""
    V, H, B, T = 200, 32768, 3, 3
    gen = torch.Generator(device="cuda").manual_seed(4)
    draw = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    E, Wo, b = draw(V, H) * 0.1, draw(V, H) * 0.01, draw(V)
    U = draw(H, H) * 0.005
    x, y = dev(tokens(V, T * B, 21).reshape(T, B)), dev(tokens(V, T * B, 22).reshape(T, B))
    m = binding.Rnnlm(E, U, Wo, b, B, T, BF16)
    r = m.rnnlm_grad_chunk(x, y)
    m.rnnlm_check()
    m.close()
    E, U, Wo, b = (t.double() for t in (E, U, Wo, b))
    h = [torch.zeros(B, H, dtype=torch.float64, device="cuda")]
    for t in range(T):
        h.append(torch.sigmoid(E[x[t].long()] + h[-1] @ U.t()))
    z = torch.stack(h[1:]) @ Wo.t() + b
    logp = z.log_softmax(2)
    dz = (logp.exp() - torch.nn.functional.one_hot(y.long(), V)) / (B * T)
    da, dU, dE = torch.zeros_like(h[0]), torch.zeros_like(U), torch.zeros_like(E)
    for t in reversed(range(T)):
        da = (dz[t] @ Wo + da @ U) * h[t + 1] * (1 - h[t + 1])
        dU += da.t() @ h[t]
        dE.index_add_(0, x[t].long(), da)
    want = dict(gE=dE, gU=dU, gWo=(dz.reshape(T * B, V).t() @ torch.cat(h[1:])), gb=dz.sum((0, 1)))
    assert (r["logp"] - logp.gather(2, y.long()[..., None])[..., 0]).abs().max() < 2e-2
    for k, w in want.items():
        assert (r[k] - w).norm() <= 2e-2 * w.norm(), k


def test_late_workgroups_are_waited_for():
    """Another stream's kernel holds a compute unit (a scan along the rows of one block of columns, some 0.2 s) while a
    window starts whose recurrent kernel wants all of them: its last workgroup starts when the scan is over, the others
    wait for it within the default limit of about a second, and the window is scored as on an idle device."""
    V, H, B, T = 500, 2048, 256, 6
    E, U, Wo, b = synth.make_weights(V, H, "normal", 0.02, 3)
    x = dev(tokens(V, T * B, 11).reshape(T, B))
    y = dev(tokens(V, T * B, 12).reshape(T, B))
    m = binding.Rnnlm(E, U, Wo, b, B, T, BF16)
    want = m.rnnlm_forward_logprob(x, y).clone()
    m.rnnlm_check()
    m.rnnlm_reset_state()
    rows = torch.zeros(400000, 512, device="cuda")
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        held = torch.cumsum(rows, 0)
    got = m.rnnlm_forward_logprob(x, y)
    m.rnnlm_check()
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    del held


@pytest.mark.parametrize("precision,H,B", [(BF16, 1024, 128), (BF16, 700, 256), (FP32, 512, 256), (FP32, 300, 200)])
def test_two_handles_train_side_by_side(precision, H, B):
    """Windows of two handles on streams of their own overlap, at the largest shapes the header allows: the workgroups of two
    recurrent kernels fit the device together, however they are dispatched.  Both handles end up with the weights that
    each trains to alone."""
    V, T, K = 300, 6, 60
    E, U, Wo, b = synth.make_weights(V, H, "normal", 0.03, 3)
    x = dev(tokens(V, K * T * B, 31).reshape(K, T, B))
    y = dev(tokens(V, K * T * B, 32).reshape(K, T, B))

    def train(models, streams):
        torch.cuda.synchronize()
        for k in range(K):
            for m, s in zip(models, streams):
                m.rnnlm_train_chunk(x[k], y[k], 0.05, stream=s)
        torch.cuda.synchronize()
        for m in models:
            m.rnnlm_check()

    alone = binding.Rnnlm(E, U, Wo, b, B, T, precision)
    train([alone], [torch.cuda.current_stream()])
    pair = [binding.Rnnlm(E, U, Wo, b, B, T, precision) for _ in range(2)]
    train(pair, [torch.cuda.Stream(), torch.cuda.Stream()])
    for m in pair:
        for n in ("E", "U", "Wo", "b", "h_state"):
            assert torch.equal(getattr(m, n), getattr(alone, n)), n
