"""bf16 contractions on 256 x 256, 128 x 128 and 64 x 64 output tiles: windows at the edges of the tiles, where an estimate of
the time chooses between them and pads positions and units to as little as the tile asks for; windows whose updates share a launch."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1502_00512_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
binding = pytest.importorskip("paper_1502_00512_amd.binding")


@pytest.mark.parametrize("V,H,B,T", [
    (257, 63, 1, 1),      # one position, one tile row past a multiple
    (1000, 65, 5, 13),    # 65 positions and 65 units: one past the smallest tile
    (3001, 200, 7, 11),   # 77 positions, padded to 128
    (3000, 129, 43, 3),   # 129 positions and units
    (9000, 384, 32, 8),   # 256 positions exactly
    (700, 500, 96, 20),   # few words, long window: many positions per tile of words
    (12000, 300, 60, 16), # 128 x 128 tiles, units past a multiple of 256
    (200, 64, 1024, 70),  # 71680 positions over one row of output tiles
])
def test_bf16_window_against_oracle(V, H, B, T):
    E, U, Wo, b = synth.make_weights(V, H, "normal", 0.05, 911 + V)
    tok = synth.zipf_tokens(2 * B * T + B + 1, V, 1.05, 37)
    g = binding.Rnnlm(E, U, Wo, b, B, T, binding.RNNLM_BF16_FP32MASTER)
    o = O.Model.from_weights(E, U, Wo, b, B)
    for k, Tn in ((0, T), (1, max(1, T // 2))):  # the shorter window has its own tiles, in the same workspace
        x, y = O.stream_chunk(tok, B, Tn, k)
        got = g.rnnlm_grad_chunk(torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda())
        ref = O.grad_chunk(o, x, y)
        # the bounds of the suite for bf16: 2e-2 of each tensor's scale (8 significant bits, a length-H dot product)
        for key in ("logp", "gE", "gU", "gWo", "gb"):
            a = got[key].cpu().numpy().astype(np.float64)
            assert np.abs(a - ref[key]).max() <= 2e-2 * np.abs(ref[key]).max(), key


@pytest.mark.parametrize("precision", [binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER])
@pytest.mark.parametrize("V,H,B,T", [
    (40, 300, 64, 16),    # 1024 positions, runs of equal ids beyond what one wave sums, two column blocks
    (30, 1100, 5, 13),    # 65 positions, more column blocks than a workgroup has waves
    (5000, 70, 8, 8),     # 64 positions: the last window on the fp32 cores; ragged rows
    (20000, 130, 3, 50),  # 128 x 128 tiles
    (700, 64, 1, 1),
])
def test_updates_in_one_launch(V, H, B, T, precision):
    E, U, Wo, b = synth.make_weights(V, H, "uniform", 0.1, 5 + V)
    tok = synth.zipf_tokens(B * T + B + 1, V, 1.05, 3)
    g = binding.Rnnlm(E, U, Wo, b, B, T, precision)
    o = O.Model.from_weights(E, U, Wo, b, B)
    x, y = O.stream_chunk(tok, B, T, 0)
    before = {n: getattr(o, n).copy() for n in ("E", "U", "Wo", "b")}
    g.rnnlm_train_chunk(torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda(), 0.5)
    O.train_chunk(o, x, y, 0.5)
    g.rnnlm_check()
    # the suite's bounds for gradients, on what the step moved: 1e-3 of each tensor's largest entry in fp32, 2e-2 in bf16;
    # the weights themselves are kept in fp32 (half an ulp of weights up to 0.6: 3e-8)
    tol = 1e-3 if precision == binding.RNNLM_FP32 else 2e-2
    for name, old in before.items():
        got, ref = getattr(g, name).cpu().numpy().astype(np.float64), getattr(o, name)
        assert np.abs(got - ref).max() <= tol * np.abs(ref - old).max() + 6e-8, name
    untouched = np.setdiff1d(np.arange(V), x)
    assert np.array_equal(g.E.cpu().numpy()[untouched], E[untouched])



@pytest.mark.parametrize("precision", [binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER])
@pytest.mark.parametrize("V,H,P,B,T", [(1000, 64, 0, 4, 8), (30, 1100, 0, 5, 13), (20000, 130, 0, 3, 50), (5000, 70, 0, 40, 16),
                                       (3000, 300, 100, 16, 9)])
def test_timed_stages_of_short_windows(V, H, P, B, T, precision):
    """Every stage of a window is executed once and takes time, and the window's results are those of an untimed one."""
    rng = np.random.default_rng(V)
    w = lambda *s: rng.uniform(-0.1, 0.1, s).astype(np.float32)
    args, more = [w(V, P or H), w(H, H), None if P else w(V, H), w(V)], dict(A=w(H, P), C_=w(P, H)) if P else {}
    f, g = binding.Rnnlm(*args, B, T, precision, **more), binding.Rnnlm(*args, B, T, precision, **more)
    x, y = (torch.as_tensor(a).cuda() for a in O.stream_chunk(synth.zipf_tokens(B * T + B + 1, V, 1.05, 3), B, T, 0))
    f.rnnlm_train_chunk(x, y, 0.5)
    g.rnnlm_profile_enable((1 << len(binding.STAGES)) - 1)
    g.rnnlm_train_chunk(x, y, 0.5)
    for name in ("stats", "softmax_grad", "out_bwd_w", "rec_w", "emb"):
        ms, executions = g.rnnlm_profile_read(binding.STAGES.index(name))
        assert executions == 1 and ms > 0, name
    g.rnnlm_profile_enable(0)
    old = dict(E=args[0], U=args[1], b=args[3], **(dict(A=more["A"], C=more["C_"]) if P else dict(Wo=args[2])))
    for name, before in old.items():
        a, b = getattr(g, name), getattr(f, name)
        # equal but for the order in which a very short window's statistics are added up: log-sums a few ulps of 2^-24 apart,
        # of 10 at most, and in bf16 gradients that then round to the other side here and there (2^-9 of an entry; the
        # weights are kept in fp32, half an ulp of values up to 0.6)
        tol = 1e-5 if precision == binding.RNNLM_FP32 else 4e-3
        moved = (b - torch.as_tensor(before).cuda()).abs().max().item()
        assert (a - b).abs().max().item() <= tol * moved + 6e-8, name
    f.rnnlm_check()
    g.rnnlm_check()


@pytest.mark.parametrize("precision", [binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER])
@pytest.mark.parametrize("V,H,P,B,T,windows", [
    (3000, 64, 0, 4, 5, 101),     # many windows a pass, one left over
    (3000, 64, 0, 3, 7, 2),
    (9000, 300, 0, 20, 10, 17),
    (2000, 200, 100, 6, 9, 40),   # compressed architecture
    (300, 500, 0, 9, 4, 5),       # the logits' space holds hardly more than a window
    (3000, 1100, 0, 2, 3, 4),     # fp32: one window at a time
])
def test_perplexity_of_long_texts(V, H, P, B, T, windows, precision):
    rng = np.random.default_rng(V + H)
    w = lambda *s: rng.uniform(-0.1, 0.1, s).astype(np.float32)
    args = [w(V, P or H), w(H, H), None if P else w(V, H), w(V)]
    more = dict(A=w(H, P), C_=w(P, H)) if P else {}
    tok = synth.zipf_tokens(windows * B * T + B + 1, V, 1.05, 3)
    a = binding.Rnnlm(*args, B, T, precision, **more)
    b = binding.Rnnlm(*args, B, T, precision, **more)
    dtok = torch.as_tensor(tok).cuda()
    for _ in range(2):
        ppl, scored = a.rnnlm_perplexity(dtok, T)
        # the same windows one call at a time: other tiles, so other orders of the sums
        b.rnnlm_reset_state()
        total = 0.0
        for k in range(windows):
            total += b.rnnlm_forward_logprob(*b.rnnlm_stream_chunk(dtok, k, T)).double().sum().item()
        assert scored == windows * B * T
        rel = 1e-5 if precision == binding.RNNLM_FP32 else 1e-3
        assert abs(ppl - np.exp(-total / scored)) <= rel * ppl
        assert (a.h_state - b.h_state).abs().max().item() <= (1e-5 if precision == binding.RNNLM_FP32 else 1e-2)
        # and the workspace is as it was: the next windows' training is the same
        a.h_state.copy_(b.h_state)
        for k in range(2):
            for m in (a, b):
                m.rnnlm_train_chunk(*m.rnnlm_stream_chunk(dtok, k, T), 0.1)
        assert torch.equal(a.E, b.E) and torch.equal(a.U, b.U) and torch.equal(a.b, b.b)
    a.rnnlm_check()


# the inserted layers over few positions, one, two and four blocks of 16, against the same layers over the padded window
# (a window of gradients, which keeps the log-probabilities)
@pytest.mark.parametrize("V,H,P,B,T", [(500, 100, 70, 1, 1), (900, 256, 64, 2, 8), (2000, 1000, 500, 1, 20), (700, 333, 130, 9, 7)])
def test_inserted_layers_over_few_positions(V, H, P, B, T):
    rng = np.random.default_rng(V)
    w = lambda *s: rng.uniform(-0.2, 0.2, s).astype(np.float32)
    g = binding.Rnnlm(w(V, P), w(H, H), None, w(V), B, T, binding.RNNLM_BF16_FP32MASTER, A=w(H, P), C_=w(P, H))
    x = torch.as_tensor(rng.integers(0, V, (T, B)).astype(np.int32)).cuda()
    y = torch.as_tensor(rng.integers(0, V, (T, B)).astype(np.int32)).cuda()
    ref = g.rnnlm_grad_chunk_compressed(x, y)["logp"]  # (the state is left as it was)
    got = g.rnnlm_forward_logprob(x, y)
    # sums in another order before two roundings to 8 bits: a few of them, 2^-9 each, on logits of the order of 1
    assert (got - ref).abs().max().item() <= 2e-2
    g.rnnlm_check()


def compressed(V, H, P, B, T):
    rng = np.random.default_rng(V + P)
    w = lambda *s: rng.uniform(-0.2, 0.2, s).astype(np.float32)
    return binding.Rnnlm(w(V, P), w(H, H), None, w(V), B, T, binding.RNNLM_BF16_FP32MASTER, A=w(H, P), C_=w(P, H))


# P: the output layer reads the layer above the state in whole blocks of 64 units, the scores in blocks of 256
@pytest.mark.parametrize("V,H,P,B,T", [(10000, 256, 100, 1, 20), (3000, 300, 70, 3, 7), (5000, 512, 257, 2, 10)])
def test_a_short_text_after_a_long_one(V, H, P, B, T):
    """What a long text leaves in the workspace has no part in a text of up to 64 positions."""
    tok = torch.as_tensor(synth.zipf_tokens(20 * B * T + B + 1, V, 1.05, 11)).cuda()
    short = tok[:3 * B * T + B + 1].contiguous()
    g, fresh = compressed(V, H, P, B, T), compressed(V, H, P, B, T)
    for _ in range(2):
        g.rnnlm_perplexity(tok, T)
        assert g.rnnlm_perplexity(short, T) == fresh.rnnlm_perplexity(short, T)
        assert torch.equal(g.h_state, fresh.h_state)


@pytest.mark.parametrize("V,H,P,B,T", [(900, 256, 64, 2, 8), (2000, 300, 100, 1, 20), (700, 333, 257, 9, 7)])
def test_scores_after_a_window_that_diverged(V, H, P, B, T):
    """A window that is not finite leaves nothing behind once the weights and the state are finite again."""
    tok = synth.zipf_tokens(2 * B * T + B + 1, V, 1.05, 5)
    x, y = (torch.as_tensor(a).cuda() for a in O.stream_chunk(tok, B, T, 0))
    g, fresh = compressed(V, H, P, B, T), compressed(V, H, P, B, T)
    g.U[0, 0] = float("nan")
    g.rnnlm_sync_compute_copies()
    g.rnnlm_train_chunk(x, y, 0.1)
    with pytest.raises(binding.RnnlmError) as e:
        g.rnnlm_check()
    assert e.value.status == -3  # RNNLM_ERR_NONFINITE
    for name in ("E", "U", "A", "C", "b", "h_state"):
        getattr(g, name).copy_(getattr(fresh, name))
    g.rnnlm_sync_compute_copies()
    cand = torch.as_tensor(np.random.default_rng(3).integers(0, V, (T, B, 10)).astype(np.int32)).cuda()
    for call in (lambda m: m.rnnlm_forward_score(x, y), lambda m: m.rnnlm_forward_score_shortlist(x, cand),
                 lambda m: m.rnnlm_forward_logprob(x, y)):
        a, b = call(g), call(fresh)
        assert torch.isfinite(b).all() and torch.equal(a, b)
    g.rnnlm_check()
