"""GPU parity of the projections from three to 64 rows over the kernels that share them (small matrices, streaming,
vector ALUs) at their edges, against fp64 products of the same (dequantized) weights; the accumulated form against the
plain one; a first call inside a stream capture."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2609_21704_amd as sq
from paper_2609_21704_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def weights(kind, n, k):
    """The call's weight arguments and the fp64 weights they stand for."""
    w = synth.normal_f16((n, k), 0.02, synth.stream_seed(41, n, k), torch.device(DEV))
    if kind == "f16":
        return (w,), w.double()
    if kind == "fp8":
        c, s = sq.sq_quantize_fp8_e4m3(w)
        return (c, s), c.view(torch.float8_e4m3fn).double() * s.double()[:, None]
    c, s, z = sq.sq_quantize_int4_g128(w)
    q = torch.stack([c & 15, c >> 4], -1).view(n, k // 128, 128).double()
    return (c, s, z), ((q - z.double()[..., None]) * s.double()[..., None]).view(n, k)


CALL = {"f16": sq.sq_verify_gemm_f16, "int4": sq.sq_qgemv_w4a16, "fp8": sq.sq_qgemv_w8a16}
# one output row, the edges of 16-row tiles, one step of k and less, tails of a step, fewer steps than wavefronts;
# both sides of the small-matrix rule (4096 outputs or k, 640000 / 16 products a row of tiles), long rows, many rows
EDGES = [("int4", 1, 128), ("int4", 15, 256), ("int4", 33, 1152), ("fp8", 1, 16), ("fp8", 17, 144), ("fp8", 47, 2064),
         ("f16", 1, 8), ("f16", 16, 136), ("f16", 65, 1160)]
SIDES = [(kind, n, k) for kind in ("int4", "fp8", "f16")
         for n, k in ((4096, 1024), (4112, 2560), (1536, 4096), (1536, 4224), (9728, 896), (14400, 2048), (1040, 6272))]


@pytest.mark.parametrize("kind,n,k", EDGES + SIDES)
def test_projection_routes(kind, n, k):
    args, ref_w = weights(kind, n, k)
    for m in (3, 4, 5, 8, 9, 16, 17, 32, 33, 49, 64):
        x = synth.normal_f16((m, k), 1.0, synth.stream_seed(42, m, k), torch.device(DEV))
        ref = x.double() @ ref_w.t()
        # fp32 sums of k exact products in any order: k 2^-24 of their magnitudes at most (and the row scale's rounding)
        bound = (x.double().abs() @ ref_w.abs().t()) * ((k + 2) * 2.0 ** -24) + 1e-30
        y = CALL[kind](x, *args)
        assert y.dtype == torch.float32 and bool(((y.double() - ref).abs() <= bound).all()), m
        # and over all of them at fp32's own error (these sums: 1.6e-7 at most); 16 bits anywhere give 1e-4 and more
        assert float((y.double() - ref).norm() / ref.norm()) <= 3e-7, m
        half = CALL[kind](x, *args, y=torch.full((m, n), float("nan"), dtype=torch.float16, device=DEV))
        assert torch.equal(half, y.half()), m
        if kind == "int4" and m <= 8 and k * m * 2 <= 65536:
            acc = synth.normal_f32((m, n), 1.0, synth.stream_seed(43, m, n), torch.device(DEV))
            want = acc + y
            sq.sq_qgemv_w4a16_acc(x, *args, acc)
            assert torch.equal(acc, want), m


@pytest.mark.parametrize("k", [128, 640, 3584])
def test_int4_infinite_scale_of_the_last_group(k):
    """A row whose last group's scale is infinite: infinities (the group's sums are not zero) from the matrix-core
    kernels, whose steps past the row's end add nothing, and the other rows as ever."""
    n = 48
    (c, s, z), _ = weights("int4", n, k)
    s[5, -1] = float("inf")
    q = torch.stack([c & 15, c >> 4], -1).view(n, k // 128, 128).double()
    for m in (9, 16, 33, 64):
        x = synth.normal_f16((m, k), 1.0, synth.stream_seed(44, m, k), torch.device(DEV))
        last = x[:, -128:].double() @ (q - z.double()[..., None])[5, -1]
        y = sq.sq_qgemv_w4a16(x, c, s, z)
        assert bool(last.abs().min() > 0) and torch.equal(y[:, 5].double(), last * float("inf")), m
        assert bool(torch.isfinite(y[:, [i for i in range(n) if i != 5]]).all()), m


CHILD = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
import paper_2609_21704_amd as sq
from paper_2609_21704_amd import synth
w = synth.normal_f16((9728, 3584), 0.02, 5, torch.device("cuda"))
x = synth.normal_f16((8, 3584), 1.0, 6, torch.device("cuda"))
q4, q8 = sq.sq_quantize_int4_g128(w), sq.sq_quantize_fp8_e4m3(w)
ys = [torch.zeros((8, 9728), device="cuda") for _ in range(2)]
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):  # the library's workspace is still empty
    sq.sq_qgemv_w4a16(x, *q4, y=ys[0])
    sq.sq_qgemv_w8a16(x, *q8, y=ys[1])
for _ in range(3):
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(ys[0], sq.sq_qgemv_w4a16(x, *q4)) and torch.equal(ys[1], sq.sq_qgemv_w8a16(x, *q8))
    for y in ys:
        y.zero_()
print("captured first", flush=True)
"""


def test_draft_projections_captured_as_first_calls():
    res = subprocess.run([sys.executable, "-c", CHILD, ROOT], capture_output=True, text=True, timeout=110)
    assert res.returncode == 0 and "captured first" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]
