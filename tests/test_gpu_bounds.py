"""No window writes next to the caller's arrays: every master and every exported gradient lies between blocks of a known
pattern, which have to come out bit for bit as they were.  The pattern is a signalling NaN, so that an access that writes
back what it read shows as well (arithmetic quiets it).  The compute copy of the output layer is looked at entry by entry,
its padding included."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1502_00512_amd import binding, synth

pytestmark = pytest.mark.gpu

FP32, BF16 = binding.RNNLM_FP32, binding.RNNLM_BF16_FP32MASTER
PATTERN = 0x7FA5A5A5


class Fenced:
    """A float32 array in the middle of a larger allocation; more than a tile's rows of pattern on both sides."""

    def __init__(self, shape, values=None):
        n, self.fence = int(np.prod(shape)), 300 * int(shape[-1] if len(shape) > 1 else 1) + 1024
        self.fence += -self.fence % 64
        self.whole = torch.full((n + 2 * self.fence,), PATTERN, dtype=torch.int32, device="cuda")
        self.array = self.whole[self.fence:self.fence + n].view(torch.float32).view(*shape)
        self.whole[self.fence:self.fence + n] = 0
        if values is not None:
            self.array.copy_(torch.as_tensor(values))

    def intact(self):
        n = self.array.numel()
        return bool((self.whole[:self.fence] == PATTERN).all()) and bool((self.whole[self.fence + n:] == PATTERN).all())


# V against tiles of 64, 128 and 256 rows (wave tiles of 32, 64 and 128): one row and a few past the last whole tile, whole
# 32-row blocks missing behind a few, one row short; H: odd, one column past a block, whole blocks of four; long and short
# windows and vocabularies, so that each tile form of the fp32 update has its turn
@pytest.mark.parametrize("precision", [FP32, BF16])
@pytest.mark.parametrize("V,H,P,B,T", [
    (257, 65, 0, 5, 7), (264, 255, 0, 5, 40), (1000, 200, 0, 8, 3), (1001, 129, 0, 30, 30), (1055, 64, 0, 64, 2),
    (2047, 300, 0, 3, 3), (20001, 520, 0, 128, 16), (30730, 257, 0, 60, 20), (7900, 1030, 0, 100, 9), (12289, 2300, 0, 6, 5),
    (1000, 64, 33, 5, 9), (5001, 200, 260, 40, 16),
])
def test_windows_write_nothing_beside_the_callers_arrays(V, H, P, B, T, precision):
    D = P or H
    E, U, Wo, b = synth.make_weights(V, H, "uniform", 0.1, V + H)
    if P:
        rng = np.random.default_rng(V)
        E, A, Cm = (rng.uniform(-0.1, 0.1, s).astype(np.float32) for s in ((V, P), (H, P), (P, H)))
    else:
        A = Cm = None
    masters = {"E": Fenced(E.shape, E), "U": Fenced(U.shape, U), "b": Fenced(b.shape, b), "h_state": Fenced((B, H))}
    masters.update({"A": Fenced(A.shape, A), "C": Fenced(Cm.shape, Cm)} if P else {"Wo": Fenced(Wo.shape, Wo)})
    lib = binding.load()
    cfg = binding.rnnlm_config(V, H, B, T, precision, 0, 0, 0, P)
    ws = torch.empty(int(lib.rnnlm_workspace_bytes(C.byref(cfg))), dtype=torch.uint8, device="cuda")
    ptr = lambda n: masters[n].array.data_ptr() if n in masters else None
    buf = binding.rnnlm_buffers(ptr("E"), ptr("U"), ptr("Wo"), ptr("b"), ptr("h_state"), ws.data_ptr(), ws.numel(),
                                ptr("A"), ptr("C"))
    h, st = C.c_void_p(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert lib.rnnlm_init(C.byref(cfg), C.byref(buf), C.byref(h)) == 0
    try:
        tok = synth.zipf_tokens(B * T + B + 1, V, 1.1, 6)
        x, y = (torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in O.stream_chunk(tok, B, T, 0))
        dv = lambda t: C.c_void_p(t.data_ptr())
        shapes = [(V, D)] + ([(H, P), (H, H), (P, H)] if P else [(H, H), (V, H)]) + [(V,)]
        grads = [Fenced(s) for s in shapes]
        export = lib.rnnlm_grad_chunk_compressed if P else lib.rnnlm_grad_chunk
        assert export(h, dv(x), dv(y), T, *[dv(g.array) for g in grads], None, st) == 0
        assert lib.rnnlm_check(h, st) == 0
        for s, g in zip(shapes, grads):
            assert g.intact(), s
            assert bool(torch.isfinite(g.array).all()), s
        assert lib.rnnlm_train_chunk(h, dv(x), dv(y), T, 0.5, None, None, st) == 0
        assert lib.rnnlm_check(h, st) == 0
        for n, m in masters.items():
            assert m.intact(), n
            assert bool(torch.isfinite(m.array).all()), n
        # the workspace begins with the compute copy of the output layer's matrix: rows and columns padded to 256 with zeros
        Vp, Dp = -(-V // 256) * 256, -(-D // 256) * 256
        dt, es = (torch.float32, 4) if precision == FP32 else (torch.bfloat16, 2)
        copy = ws[:Vp * Dp * es].view(dt).view(Vp, Dp)
        assert torch.equal(copy[:V, :D], masters["E" if P else "Wo"].array.to(dt))
        assert not bool(copy[V:].any()) and not bool(copy[:, D:].any())
    finally:
        torch.cuda.synchronize()
        lib.rnnlm_free(h)
