"""GPU checks of the prefill calls (include/specquant_prefill.h): projections at any number of rows against fp64
products of the same (dequantized) weights, in all three output forms; the rotation against sq_rope_kv_f16 in blocks of
64 (the same bits); the attention against the oracle; a whole prompt against the same prompt in blocks of 64."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21704_amd as sq
from paper_2609_21704_amd import _lib as lib
from paper_2609_21704_amd import decoder as dec
from paper_2609_21704_amd import synth
from paper_2609_21704_amd.configs import Config

pytestmark = pytest.mark.gpu
DEV = "cuda"


def weights(kind, n, k, seed):
    """The call's weight arguments and the fp64 weights they stand for."""
    w = synth.normal_f16((n, k), 0.02, synth.stream_seed(seed, n, k), torch.device(DEV))
    if kind == "f16":
        return (w,), w.double()
    if kind == "fp8":
        c, s = sq.sq_quantize_fp8_e4m3(w)
        return (c, s), c.view(torch.float8_e4m3fn).double() * s.double()[:, None]
    c, s, z = sq.sq_quantize_int4_g128(w)
    q = torch.stack([c & 15, c >> 4], -1).view(n, k // 128, 128).double()
    return (c, s, z), ((q - z.double()[..., None]) * s.double()[..., None]).view(n, k)


CALL = {"f16": lib.sq_prefill_linear_f16, "int4": lib.sq_prefill_linear_w4, "fp8": lib.sq_prefill_linear_w8}
# edges of the 128- and 256-row tiles and of the 256 (SiLU: 128) outputs, one step of k and more, odd outputs, K parts
SHAPES = [(1, 64, 128), (65, 77, 640), (128, 256, 256), (129, 258, 384), (257, 514, 384), (100, 4608, 1024),
          (300, 1000, 3584), (511, 2050, 2048), (2000, 512, 1152)]
# tiles of 192 and 256 rows (FP16 and FP8 over 256 CUs), whole rows of even and odd steps, and K parts, ragged in rows
# and outputs
TALL = [(1547, 5042, 320), (1547, 5041, 128), (1993, 5978, 320), (1995, 5982, 128), (161, 5574, 2688), (152, 5430, 4032),
        (387, 5674, 2432), (398, 5526, 4480)]


@pytest.mark.parametrize("kind", ["f16", "fp8", "int4"])
@pytest.mark.parametrize("m,n,k", SHAPES + TALL + [(130, 96, 64), (70, 300, 192)])
def test_prefill_linear(kind, m, n, k):
    if kind == "int4" and k % 128:
        return
    args, ref_w = weights(kind, n, k, 31)
    x = synth.normal_f16((m, k), 1.0, synth.stream_seed(32, m, k), torch.device(DEV))
    ref = x.double() @ ref_w.t()
    # fp32 sums of k exact products in any order: k 2^-24 of their magnitudes at most
    bound = (x.double().abs() @ ref_w.abs().t()) * (k * 2.0 ** -24) + 1e-30
    y = torch.full((m, n), float("nan"), device=DEV)
    assert CALL[kind](x, *args, y)
    assert bool(((y.double() - ref).abs() <= bound).all())
    # and over all of them at fp32's own error (these sums: 1.5e-7 at most); 16 bits anywhere give 1e-4 and more
    assert float((y.double() - ref).norm() / ref.norm()) <= 3e-7
    base = synth.normal_f32((m, n), 1.0, synth.stream_seed(33, m, n), torch.device(DEV))
    acc = base.clone()
    assert CALL[kind](x, *args, acc, lib.PREFILL_ADD)
    # the same product, added: one more fp32 rounding (K parts add it to the base in the same order)
    assert bool(((acc.double() - base.double() - ref).abs() <= bound + 2.0 ** -23 * (base.double() + ref).abs()).all())
    assert torch.equal(acc, base + y)
    if n % 2 == 0:
        t = torch.full((m, n // 2), float("nan"), dtype=torch.float16, device=DEV)
        assert CALL[kind](x, *args, t, lib.PREFILL_SILU)
        g, u = ref.chunk(2, 1)
        want = g * torch.sigmoid(g) * u
        tol = 2.0 ** -10 * want.abs() + 4 * (bound[:, :n // 2] * (u.abs() + 1) + bound[:, n // 2:] * (g.abs() + 1)) + 1e-7
        assert bool(((t.double() - want).abs() <= tol).all())


# Relative errors (2-norm, in 1e-7) of sums in blocks and of the blocks, as the streaming kernel for 64 rows forms them:
# 0.51 .. 2.29 for these kinds and row lengths, and a tenth more.  One running sum gives 1.3 to 3 times as much from
# 1536 k on.
ROUNDINGS = {"f16": {896: 1.21, 1536: 1.53, 3584: 1.61, 18944: 2.52}, "fp8": {896: 1.2, 1536: 1.56, 3584: 1.57, 18944: 2.01},
             "int4": {896: 0.6, 1536: 0.63, 3584: 0.76, 18944: 1.11}}


# one tile per CU and K parts, more rounds of the larger tiles, long rows
@pytest.mark.parametrize("kind", ["f16", "fp8", "int4"])
@pytest.mark.parametrize("m,n,k", [(300, 1000, 896), (2000, 2048, 1536), (2000, 4608, 3584), (2000, 3584, 3584),
                                   (2000, 3584, 18944), (4000, 3584, 18944)])
def test_prefill_linear_rounds_as_sums_in_blocks(kind, m, n, k):
    args, ref_w = weights(kind, n, k, 34)
    x = synth.normal_f16((m, k), 1.0, synth.stream_seed(35, m, k), torch.device(DEV))
    ref = x.double() @ ref_w.t()
    y = torch.empty((m, n), device=DEV)
    assert CALL[kind](x, *args, y)
    error = float((y.double() - ref).norm() / ref.norm())
    assert error <= 1e-7 * ROUNDINGS[kind][k], error


@pytest.mark.parametrize("b,rows,hq,hkv,offset", [(1, 130, 7, 1, 0), (2, 80, 4, 2, 64), (3, 65, 6, 3, 5)])
def test_prefill_rope_equals_blocks(b, rows, hq, hkv, offset):
    cap = 256
    qkv = synth.normal_f32((b * rows, (hq + 2 * hkv) * 128), 1.0, 41, torch.device(DEV))
    bias = synth.normal_f16(((hq + 2 * hkv) * 128,), 0.5, 42, torch.device(DEV))
    pos = torch.tensor([0, 3, 90][:b], dtype=torch.int32, device=DEV)  # the last sequence runs past len_bound
    lb = offset + rows + 40
    caches = [[torch.zeros((b, hkv, cap, 128), dtype=torch.float16, device=DEV),
               torch.zeros((b, hkv, 128, cap), dtype=torch.float16, device=DEV)] for _ in range(2)]
    st = [torch.zeros(1, dtype=torch.int32, device=DEV) for _ in range(2)]
    q = lib.sq_prefill_rope_kv_f16(qkv, bias, pos, offset, rows, hq, *caches[0], len_bound=lb, status=st[0])
    view = qkv.view(b, rows, -1)
    for s in range(0, rows, 64):
        n = min(64, rows - s)
        qb = sq.sq_rope_kv_f16(view[:, s:s + n].reshape(b * n, -1).contiguous(), bias, pos, offset + s, n, hq, *caches[1],
                               len_bound=lb, status=st[1])
        assert torch.equal(q.view(b, rows, hq, 128)[:, s:s + n].reshape(b * n, hq, 128).view(torch.int16),
                           qb.view(torch.int16))
    assert all(torch.equal(a.view(torch.int16), c.view(torch.int16)) for a, c in zip(*caches))
    assert torch.equal(st[0], st[1])


@pytest.mark.parametrize("rows,hq,hkv,p0,cap", [(65, 7, 1, 0, 128), (100, 4, 2, 37, 192), (200, 3, 3, 0, 256)])
def test_prefill_attention_matches_the_oracle(rows, hq, hkv, p0, cap):
    q = synth.normal_f16((rows, hq, 128), 1.5, 51)
    kc, vc = synth.normal_f16((1, hkv, cap, 128), 1.0, 52), synth.normal_f16((1, hkv, 128, cap), 1.0, 53)
    end = p0 + rows
    kc[:, :, end:] = float("nan")  # entries past the block: never read
    vc[:, :, :, end:] = float("nan")
    pos = torch.tensor([p0], dtype=torch.int32, device=DEV)
    out = lib.sq_prefill_attention_f16(q.to(DEV), kc.to(DEV), vc.to(DEV), pos, 0, rows)
    vv = np.swapaxes(vc[0, :, :, :end].double().numpy(), 1, 2)
    ref = oracle.attention(q.double().numpy(), kc[0, :, :end].double().numpy(), vv, np.arange(p0, end))
    assert np.abs(out.cpu().double().numpy() - ref).max() <= 2e-3 * np.abs(vv).max()


@pytest.mark.parametrize("variant,batch,chains,lengths", [("int4", 1, 1, [130]), ("fp8", 3, 1, [90, 41, 64]),
                                                          ("int4", 2, 2, [70, 33])])
def test_prompt_in_one_pass_and_in_blocks(variant, batch, chains, lengths):
    cfg = Config(0, "prefill", 3, 512, 1152, 4, 2, 1000, variant, 2, batch, 5)
    lp = max(lengths)
    prompt = dec.synthetic_prompt(cfg, batch, lp, DEV)
    w = dec.DecoderWeights(cfg, DEV)
    a, b = (dec.SpecDecoder(w, capacity=192, chains=chains) for _ in range(2))
    a.prefill(prompt, lengths=lengths)
    b.prefill(prompt, chunk=64 // (batch * chains), lengths=lengths)
    assert int(a.status.item()) == int(b.status.item()) == 0
    for x, y in ((a.dcache, b.dcache), (a.pcache, b.pcache)):
        for u, v in ((x.k_all, y.k_all), (x.v_all, y.v_all)):
            # fp16 activations between the layers: a few of their roundings differ with the order of the sums
            assert float((u.double() - v.double()).norm() / v.double().norm()) <= 2e-3
    assert torch.equal(a.pending, b.pending) and torch.equal(a.prev, b.prev) and torch.equal(a.pos_base, b.pos_base)
