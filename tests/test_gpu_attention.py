"""GPU checks of the block attention where its kernels change path: chunks every row reads and chunks with a mask, one
to four query tiles, slots of one and of several chunks (both sides of the workgroup counts), blocks that start, end and
cross a chunk; the rotating call against the separate calls; the rotation's own exponential, cosine and sine."""
import numpy as np
import pytest
import torch

import paper_2609_21704_amd as sq
from paper_2609_21704_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def normal(shape, *seed):
    return synth.normal_f16(shape, 1.0, synth.stream_seed(51, *seed), torch.device(DEV))


# (b, rows, hq, hkv, capacity, first positions)
CASES = [(2, 1, 4, 4, 128, (63, 64)), (2, 5, 28, 4, 192, (0, 62)), (1, 9, 28, 4, 4096, (4080,)),
         (3, 16, 8, 2, 1024, (47, 48, 600)), (4, 9, 28, 4, 2112, (2000, 2039, 2047, 2048)),
         (8, 1, 28, 4, 1088, (1, 64, 65, 127, 1000, 1023, 1024, 1087)), (1, 5, 28, 4, 8256, (8191,)),
         (4, 2, 28, 4, 4160, (4100, 31, 4095, 4158))]


@pytest.mark.parametrize("b,rows,hq,hkv,cap,first", CASES)
def test_attention_paths(b, rows, hq, hkv, cap, first):
    g = hq // hkv
    kc, vc = normal((b, hkv, cap, 128), 1, cap), normal((b, hkv, 128, cap), 2, cap)
    qkv = normal((b * rows, (hq + 2 * hkv) * 128), 3, rows).float()
    bias = normal(((hq + 2 * hkv) * 128,), 4)
    pos = torch.tensor(first, dtype=torch.int32, device=DEV)
    for s in range(b):  # entries after the block may hold anything
        kc[s, :, first[s] + rows:] = float("nan")
        vc[s, :, :, first[s] + rows:] = float("nan")
    k1, v1, k2, v2 = kc.clone(), vc.clone(), kc.clone(), vc.clone()
    q = torch.empty((b * rows, hq, 128), dtype=torch.float16, device=DEV)
    sq.sq_rope_kv_f16(qkv, bias, pos, 0, rows, hq, k1, v1, q_out=q)
    out = torch.empty((b * rows, hq, 128), dtype=torch.float16, device=DEV)
    sq.sq_attention_f16(q, k1, v1, pos, 0, rows, out=out)
    fused = torch.empty_like(out)
    assert sq.sq_rope_attention_f16(qkv, bias, pos, 0, rows, hq, k2, v2, fused)
    assert torch.equal(fused, out)
    assert torch.equal(k1.view(torch.int16), k2.view(torch.int16))
    assert torch.equal(v1.view(torch.int16), v2.view(torch.int16))
    for s in range(b):
        for j in range(rows):
            n = first[s] + j + 1
            qd = q[s * rows + j].double().view(hkv, g, 128)
            kd, vd = k1[s, :, :n].double(), v1[s, :, :, :n].double()
            p = torch.softmax(torch.matmul(qd, kd.transpose(1, 2).contiguous()) / 128 ** 0.5, -1)
            vt = vd.transpose(1, 2).contiguous()
            ref, mag = torch.matmul(p, vt), torch.matmul(p, vt.abs())
            # a score: 128 fp32 terms of exact products, scaled; its error moves every weight of the row; weights and
            # sums beside it to 2^-18; the result rounded to binary16
            dot = torch.matmul(qd.abs(), kd.abs().transpose(1, 2).contiguous()).amax(-1, keepdim=True) / 128 ** 0.5
            bound = mag * (2 * dot * 132 * 2.0 ** -24 + 2.0 ** -18) + ref.abs() * 2.0 ** -11 + 2.0 ** -25
            got = out[s * rows + j].double().view(hkv, g, 128)
            assert bool(((got - ref).abs() <= bound).all()), (s, j)


@pytest.mark.parametrize("theta", [1.0000001, 10000.0, 1e6, 1e300])
def test_rotation_against_64_bits(theta):
    cap = 1 << 18
    first = [0, 1, 1000, 65535, 131071, cap - 2]
    cache = torch.zeros((6, 1, cap, 128), dtype=torch.float16, device=DEV)
    vals = torch.zeros((6, 1, 128, cap), dtype=torch.float16, device=DEV)
    qkv = normal((12, 3 * 128), 5).float()
    q = torch.empty((12, 1, 128), dtype=torch.float16, device=DEV)
    sq.sq_rope_kv_f16(qkv, None, torch.tensor(first, dtype=torch.int32, device=DEV), 0, 2, 1, cache, vals, theta=theta,
                      q_out=q)
    x = qkv.view(12, 3, 128)[:, 0].double().cpu().numpy()
    at = np.array([p + j for p in first for j in range(2)], np.float64)
    ang = at[:, None] * np.power(theta, -np.arange(64) / 64.0)
    a, e, c, s = x[:, :64], x[:, 64:], np.cos(ang), np.sin(ang)
    ref = np.concatenate([a * c - e * s, e * c + a * s], 1)
    got = q[:, 0].double().cpu().numpy()
    # fp32 cosine, sine, products and their difference, then binary16; the angles of two libraries 2^-51 of 2^18 apart
    mag = np.concatenate([np.abs(a) + np.abs(e)] * 2, 1)
    assert (np.abs(got - ref) <= mag * 2.0 ** -22 + mag * 2.0 ** -33 + np.abs(ref) * 2.0 ** -11 + 2.0 ** -25).all()
