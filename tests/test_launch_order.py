"""What calls enqueue and in which order, without a GPU: the library runs against a HIP runtime that logs launches,
event records and event waits (launch_log.cpp), and the happens-before relation between launches is rebuilt from the log.
Nothing is computed; device addresses are made up and never followed."""
import os
import re
import subprocess
import sys

import pytest

from paper_1502_00512_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))
STREAM = 0x5000
FP32, BF16 = 0, 1

# (ctypes alone: torch would bring the real runtime along)
DRIVER = """
import ctypes as C, sys
C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
lib.rnnlm_workspace_bytes.restype = C.c_size_t
call, args = sys.argv[3], eval(sys.argv[4])
cfg = (C.c_int32 * 9)(*[args[k] for k in ("V", "H", "B", "T_max", "precision")], 0, args.get("K", 0), args.get("rmsprop", 0), args.get("P", 0))
at = [1 << 44]
def dev():
    at[0] += 1 << 40
    return at[0]
class Buffers(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("E", "U", "Wo", "b", "h", "ws")] + [("bytes", C.c_size_t), ("A", C.c_void_p), ("C", C.c_void_p)]
buf = Buffers(dev(), dev(), dev(), dev(), dev(), dev(), lib.rnnlm_workspace_bytes(cfg), None, None)
if args.get("P"):
    buf.Wo, buf.A, buf.C = None, dev(), dev()
h = C.c_void_p()
assert lib.rnnlm_init(cfg, C.byref(buf), C.byref(h)) == 0
f, p, x, y, st, T = C.c_float, C.c_void_p, C.c_void_p(dev()), C.c_void_p(dev()), C.c_void_p(int(sys.argv[5])), args["T"]
rms = (C.c_void_p * 4)(dev(), dev(), dev(), dev())
noise, lnq = C.c_void_p(dev()), C.c_void_p(dev())
lib.rnnlm_profile_enable(h, args.get("profile", 0))
for _ in range(2):
    if call == "train":
        rc = lib.rnnlm_train_chunk(h, x, y, T, f(0.1), None, None, st)
    elif call == "rmsprop":
        rc = lib.rnnlm_train_chunk_rmsprop(h, x, y, T, f(0.1), f(0.9), f(1e-6), rms, None, None, st)
    elif call == "nce_rmsprop":
        rc = lib.rnnlm_nce_train_chunk_rmsprop(h, x, y, T, noise, args["K"], lnq, f(7.0), f(0.1), f(0.9), f(1e-6), rms, None, None, st)
    elif call == "logprob":
        rc = lib.rnnlm_forward_logprob(h, x, y, T, p(dev()), st)
    elif call == "perplexity":
        rc = lib.rnnlm_perplexity(h, x, C.c_int64(args["N"]), T, C.byref(C.c_double()), None, st)
    assert rc == 0, rc
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        from paper_1502_00512_amd.build import build
        build()
    so = str(tmp_path_factory.mktemp("runtime") / "liblaunch_log.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_log.cpp")], check=True)
    return so


def enqueue(runtime, tmp_path, call, **args):
    """Two calls; returns their launches as (stream, kernel, words) and before(i, j): launch i is ordered before launch j."""
    log = str(tmp_path / "log")
    r = subprocess.run([sys.executable, "-c", DRIVER, runtime, binding.LIB_PATH, call, repr(args), str(STREAM)],
                       env=dict(os.environ, LAUNCH_LOG=log), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    launches, seen, events = [], {}, {}  # seen[stream]: launches that whatever comes next on it is ordered behind
    known = []
    for line in open(log):
        op, stream, rest = line.split(None, 2)
        past = seen.setdefault(stream, set())
        if op == "L":
            kernel, *words = rest.split()
            known.append(set(past))
            past.add(len(launches))
            launches.append((int(stream, 16) if stream != "(nil)" else 0, kernel, [int(w, 16) for w in words if w != "|"]))
        elif op == "R":
            events[rest.strip()] = set(past)
        else:
            past |= events[rest.strip()]
    return launches, lambda i, j: i in known[j]


@pytest.mark.parametrize("call", ["rmsprop", "nce_rmsprop"])
@pytest.mark.parametrize("precision", [FP32, BF16])
@pytest.mark.parametrize("H", [64, 1024, 3840, 3841, 4096])  # from 3841 on the recurrent gradient is formed last
def test_rmsprop_steps_the_recurrent_matrix_behind_its_gradient(runtime, tmp_path, call, precision, H):
    launches, before = enqueue(runtime, tmp_path, call, V=3000, H=H, B=16, T_max=4, T=4, precision=precision, rmsprop=1, K=64)
    steps = [i for i, (_, k, _) in enumerate(launches) if "rms_square_apply" in k]
    assert len(steps) == 2
    gradient = launches[steps[0]][2][0]
    formed = [i for i, (_, k, w) in enumerate(launches) if "gemm" in k and gradient in w]
    assert len(formed) == 2 and formed[0] < steps[0] < formed[1] < steps[1]
    for f, s in zip(formed, steps):
        assert before(f, s)
    assert before(steps[0], formed[1])  # and the next window's is formed behind the step that read this one's


@pytest.mark.parametrize("call,H", [("train", 64), ("train", 1024), ("train", 4096), ("rmsprop", 256), ("rmsprop", 4096),
                                    ("nce_rmsprop", 256), ("nce_rmsprop", 4096)])
def test_the_callers_stream_is_behind_all_work_of_a_call(runtime, tmp_path, call, H):
    launches, before = enqueue(runtime, tmp_path, call, V=3000, H=H, B=16, T_max=4, T=4, precision=BF16, K=64,
                               rmsprop=int("rmsprop" in call))
    starts = [i for i, (_, k, _) in enumerate(launches) if "prep_tokens" in k]  # (the second call's decay comes before its)
    assert len(starts) == 2 and launches[starts[1]][0] == STREAM
    for i in range(starts[0], starts[1]):
        assert before(i, starts[1]) or "rms_decay" in launches[i][1], launches[i]


@pytest.mark.parametrize("call", ["rmsprop", "nce_rmsprop"])
@pytest.mark.parametrize("V,H,B,T,beside", [(1000, 64, 1, 1, False), (1375, 384, 4, 3, False), (64000, 1024, 128, 20, True)])
def test_rmsprop_steps_leave_the_callers_stream_in_long_windows_only(runtime, tmp_path, call, V, H, B, T, beside):
    """Every pair of events that ties the second stream in costs a short window, which the host bounds, some 10 us."""
    launches, _ = enqueue(runtime, tmp_path, call, V=V, H=H, B=B, T_max=T, T=T, precision=BF16, rmsprop=1, K=64)
    assert {s != STREAM for s, k, _ in launches if "rms_decay" in k or "rms_square_apply" in k} == {beside}


@pytest.mark.parametrize("V,H,B,T_max,T,precision", [
    (20000, 1000, 65536, 33, 1, FP32),  # 2^21 positions and more: 256 rows of the logits span 2^31 bytes
    (20000, 1000, 65536, 33, 33, FP32),
    (200, 8, 65536, 129, 1, FP32),   # 2^23: 64 rows
    (300, 40, 65536, 256, 3, FP32),  # the most positions a handle may have
    (300, 300, 65536, 256, 256, FP32),
    (200, 32768, 2, 4, 3, BF16),     # a state-to-state matrix of 2^31 bytes, few streams and whole blocks of 256
    (200, 33000, 256, 4, 3, BF16),
    (200, 33000, 3, 4, 3, FP32),
])
def test_sizes_beyond_32_bit_offsets_are_taken(runtime, tmp_path, V, H, B, T_max, T, precision):
    """Operands whose bytes a contraction kernel's 32-bit offsets do not reach take another kernel."""
    launches, _ = enqueue(runtime, tmp_path, "train", V=V, H=H, B=B, T_max=T_max, T=T, precision=precision)
    assert sum("gemm" in k for _, k, _ in launches) >= 6


@pytest.mark.parametrize("V,H,P,B,T_max,T", [
    (200, 8, 0, 1, 1 << 24, 1),      # 32 rows of the logits span 2^31 bytes
    (200, 8, 0, 1, 1 << 24, 3),
    (256, 64, 0, 32, 1 << 19, 4),
    (200, 64, 0, 1, 1 << 24, 500),
    (300, 64, 0, 1, 1 << 24, 2560),
    (700, 300, 0, 1, 1 << 24, 128),
    (1604, 400, 0, 3, (1 << 24) // 3, 100000),
    (2000, 256, 0, 1, 1 << 23, 3000),  # 64 rows
    (2000, 256, 0, 1, (1 << 23) - 256, 3000),
    (2000, 256, 100, 1, 1 << 23, 3000),
    (200, 64, 64, 1, 1 << 24, 3),
    (700, 300, 300, 1, 1 << 24, 2560),
])
def test_the_contraction_over_the_vocabulary_reaches_long_rows_of_logits(runtime, tmp_path, V, H, P, B, T_max, T):
    """fp32 handles of millions of positions: blocks of 32 or 64 rows of the logits are beyond 32-bit offsets."""
    launches, _ = enqueue(runtime, tmp_path, "train", V=V, H=H, P=P, B=B, T_max=T_max, T=T, precision=FP32)
    assert sum("gemm" in k for _, k, _ in launches) >= 6


@pytest.mark.parametrize("call", ["train", "logprob", "perplexity"])
@pytest.mark.parametrize("V,H,P,B,T_max,T", [
    (256, 64, 0, 1024, 70, 70), (2, 72, 0, 1869, 46, 46), (200, 300, 0, 257, 256, 256), (256, 512, 0, 2048, 33, 33),
    (22, 90, 0, 288, 1000, 300), (127, 100, 40, 2300, 100, 100), (256, 64, 0, 1024, 64, 64),
])
def test_long_windows_over_few_words_are_taken(runtime, tmp_path, call, V, H, P, B, T_max, T):
    """bf16, one row of 256 x 256 output tiles and more than a round of them, whole rounds or not."""
    launches, _ = enqueue(runtime, tmp_path, call, V=V, H=H, P=P, B=B, T_max=T_max, T=T, precision=BF16, N=3 * B * T + B + 1)
    assert sum("EpiOutFwd" in k for _, k, _ in launches) >= 2


@pytest.mark.parametrize("V,H,P,B,T_max,T", [
    (1604, 3659, 0, 234, 29, 29), (2920, 3338, 0, 151, 28, 28), (3209, 852, 0, 512, 44, 32), (38708, 1702, 0, 1024, 256, 256),
    (1200, 2000, 0, 256, 32, 32), (6000, 1702, 512, 512, 64, 64), (64000, 1024, 0, 128, 10, 10), (100000, 512, 0, 2048, 32, 32),
])
def test_long_sums_over_the_vocabulary_keep_their_lesser_products_apart(runtime, tmp_path, V, H, P, B, T_max, T):
    """The 256 x 256 form adds all six products of an fp32 contraction to one accumulator."""
    launches, _ = enqueue(runtime, tmp_path, "train", V=V, H=H, P=P, B=B, T_max=T_max, T=T, precision=FP32)
    # (template arguments: tile, waves, then both operands' layouts, 1 = K-major)
    over = [k for _, k, _ in launches if re.search(r"gemm_split_kernelI(?:Li\d+E){5}Li1ELi1E.*EpiPartial", k)]
    assert len(over) == 2 and not any("ILi256ELi256E" in k for k in over), over


@pytest.mark.parametrize("V,H,B,T,precision", [(3000, 4096, 256, 8, BF16), (3000, 3841, 64, 20, BF16), (3000, 4000, 64, 3, FP32)])
def test_timing_the_widest_output_update_delays_it_behind_nothing(runtime, tmp_path, V, H, B, T, precision):
    """No event lies between the fork of the embedding update and the launch of the large one, which is to come first."""
    enqueue(runtime, tmp_path, "train", V=V, H=H, B=B, T_max=T, T=T, precision=precision, profile=1 << 7)
    lines = [l.split() for l in open(tmp_path / "log")]
    own = [l for l in lines if l[1] == hex(STREAM)]
    forks = {l[2] for l in lines if l[0] == "W" and l[1] != hex(STREAM)}
    updates = [i for i, l in enumerate(own) if l[0] == "L" and "gemm" in l[2] and "EpiSgdI" in l[2]]
    assert len(updates) == 2
    for i in updates:
        assert own[i - 1][0] == "R" and own[i - 1][2] in forks  # the fork
        assert own[i - 2][0] == "R" and own[i + 1][0] == "R"    # the stage's pair around both


def timed_launches(runtime, tmp_path, stage, **args):
    """Kernels between the two events of every execution of a stage of two training calls, and all kernels."""
    launches, _ = enqueue(runtime, tmp_path, "train", profile=1 << stage, **args)
    lines = [l.split() for l in open(tmp_path / "log")]
    ordering = {l[2] for l in lines if l[0] == "W"}
    pairs, is_open = [], {}
    for op, stream, what, *_ in lines:
        if op == "L":
            for inside in is_open.values():
                inside.append(what)
        elif op == "R" and what not in ordering:
            if stream in is_open:
                pairs.append(is_open.pop(stream))
            else:
                is_open[stream] = []
    assert not is_open
    return pairs, [k for _, k, _ in launches]


STATS, SOFTMAX_GRAD, OUT_BWD_W, REC_W, EMB, PROJ = 3, 4, 7, 8, 9, 17


@pytest.mark.parametrize("V,H,B,T,precision", [(1000, 64, 4, 8, FP32), (5000, 70, 8, 9, FP32), (1000, 65, 5, 13, BF16),
                                               (20000, 130, 3, 50, BF16), (3000, 300, 60, 16, BF16)])
@pytest.mark.parametrize("stage", [OUT_BWD_W, REC_W, EMB])
def test_a_timed_update_of_a_short_window_is_a_launch_of_its_own(runtime, tmp_path, stage, V, H, B, T, precision):
    pairs, kernels = timed_launches(runtime, tmp_path, stage, V=V, H=H, B=B, T_max=T, T=T, precision=precision)
    assert [["window_update" in k for k in pair] for pair in pairs] == [[True], [True]]
    assert sum("window_update" in k for k in kernels) == 6  # three updates, two calls
    untimed, _ = enqueue(runtime, tmp_path, "train", V=V, H=H, B=B, T_max=T, T=T, precision=precision)
    assert sum("window_update" in k for _, k, _ in untimed) == 2


@pytest.mark.parametrize("precision", [FP32, BF16])
@pytest.mark.parametrize("stage,kernel", [(STATS, "merge_stats"), (SOFTMAX_GRAD, "softmax_grad")])
def test_timed_statistics_of_a_very_short_window_are_a_launch_of_their_own(runtime, tmp_path, precision, stage, kernel):
    args = dict(V=1000, H=64, B=4, T_max=8, T=8, precision=precision)
    pairs, kernels = timed_launches(runtime, tmp_path, stage, **args)
    assert [[kernel in k for k in pair] for pair in pairs] == [[True], [True]]
    assert sum("merge_stats" in k for k in kernels) == 2
    untimed, _ = enqueue(runtime, tmp_path, "train", **args)
    assert not any("merge_stats" in k for _, k, _ in untimed)


@pytest.mark.parametrize("stage", [REC_W, PROJ])
def test_a_timed_recurrent_update_of_the_compressed_architecture_is_a_launch_of_its_own(runtime, tmp_path, stage):
    args = dict(V=3000, H=300, P=100, B=16, T_max=9, T=9, precision=BF16)
    pairs, kernels = timed_launches(runtime, tmp_path, stage, **args)
    recurrent = [k for k in kernels if "gemm" in k and "EpiSgdT" in k]
    assert len(recurrent) == 2 and sum("update_group" in k for k in kernels) == 2
    inside = [k for pair in pairs for k in pair]
    assert (inside == recurrent) if stage == REC_W else not set(inside) & set(recurrent)
    untimed, _ = enqueue(runtime, tmp_path, "train", **args)
    assert not any("gemm" in k and "EpiSgdT" in k for _, k, _ in untimed)
