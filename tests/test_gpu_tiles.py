"""bf16 contractions on 256 x 256, 128 x 128 and 64 x 64 output tiles: windows at the edges of the tiles, where an estimate of
the time chooses between them and pads positions and units to as little as the tile asks for."""
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
