"""Accept calls of one draft chain where their launches change shape, against the oracle: several chunks per workgroup,
greedy rows of one and of many chunks, and scratch that other calls have written before."""
import numpy as np
import pytest
import torch

import paper_2609_21704_amd as sq
from paper_2609_21704_amd import _lib
from accept_compare import check_accept
from test_gpu_parity import _accept_case, _run_accept

pytestmark = pytest.mark.gpu
DEV = "cuda"


def check(b, kd, v, temp, seed):
    draft, target, tok, u24 = _accept_case(b, kd, v, seed, temp, "uniform" if temp == 0.0 else "sampled")
    if temp == 0.0 and kd > 0:  # accepted up to a position that differs from sequence to sequence
        tok = target[:, :kd].argmax(-1).t().to(torch.int32).contiguous()
        for s in range(b):
            if s % (kd + 1) < kd:
                tok[s % (kd + 1), s] = (tok[s % (kd + 1), s] + 1) % v
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, temp, want_pq=temp > 0)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), temp, n, t,
                 q_out.cpu().numpy() if q_out is not None else None, p_out.cpu().numpy() if p_out is not None else None)
    return n


# chunks of 1024 logits over all sequences: 512 (one per workgroup), 513 (two, the last workgroup with one), more
# sequences than workgroups, several per workgroup with draws after acceptances
@pytest.mark.parametrize("b,kd,v", [(1, 0, 524288), (1, 0, 524289), (171, 0, 3000), (600, 0, 1025), (130, 2, 4097),
                                    (9, 3, 65537), (16, 1, 151936)])
def test_spec_accept_chunks_per_workgroup(b, kd, v):
    check(b, kd, v, 1.0, 300 + b + v)


# one chunk of 4096 logits and one more logit, with and without drafts; more rows than wavefronts; 65 chunks of a row
@pytest.mark.parametrize("b,kd,v", [(3, 0, 4096), (3, 0, 4097), (2, 1, 4096), (3, 15, 4097), (4, 16, 9000),
                                    (66, 64, 130), (2, 2, 262145)])
def test_spec_accept_greedy_rows(b, kd, v):
    n = check(b, kd, v, 0.0, 400 + b + v)
    if b > kd:
        assert sorted(set(n.tolist())) == list(range(kd + 1))


# rows of one chunk, read by the deciding kernel: one to four wavefronts a row, one or two steps of 1024 logits, rows
# in two passes; the first sizes past these
@pytest.mark.parametrize("b,kd,v", [(3, 1, 1), (3, 4, 1024), (6, 4, 1025), (6, 4, 3072), (6, 4, 3073), (5, 3, 4096),
                                    (9, 7, 2048), (9, 7, 2049), (10, 8, 2047), (3, 8, 2049), (17, 15, 1000),
                                    (20, 16, 1024), (20, 16, 1025), (20, 17, 777), (33, 18, 777)])
def test_spec_accept_greedy_short_rows(b, kd, v):
    n = check(b, kd, v, 0.0, 600 + b + v)
    if b > kd:
        assert sorted(set(n.tolist())) == (list(range(kd + 1)) if v > 1 else [kd])


def test_spec_accept_greedy_short_rows_ties_and_invalid():
    """The largest logit twice, in different wavefronts' parts: the smaller index; NaN, +inf and all -inf in any part."""
    b, kd, v = 8, 3, 4096
    target = torch.randn((b, kd + 1, v), generator=torch.Generator().manual_seed(9))
    target[:, :, 700] = target[:, :, 3900] = 9.0
    target[1, 2, 4095] = float("nan")
    target[2, 3, 1500] = float("inf")
    target[3, 0] = float("-inf")
    target[4, 1, 1024:] = float("-inf")
    tok = torch.full((kd, b), 700, dtype=torch.int32)
    tok[1, 5] = 3900
    n, t, _, _ = _run_accept(torch.zeros((kd, b, v)), target, tok, torch.zeros((b, kd + 1), dtype=torch.int32), 0.0)
    assert np.array_equal(n, [3, -1, -1, -1, 3, 1, 3, 3]) and np.array_equal(t, [700, -1, -1, -1, 700, 700, 700, 700])


@pytest.mark.parametrize("temp", [1.0, 0.0])
@pytest.mark.parametrize("b,kd,v", [(1, 0, 1000), (2, 4, 9000), (40, 1, 20000)])
def test_spec_accept_after_other_calls_scratch(b, kd, v, temp):
    """The library's workspace full of another call's values: nothing in it needs to be as a call left it."""
    g = torch.Generator(device=DEV).manual_seed(5)
    rows = torch.randn((2, 4, 4, 60000), generator=g, device=DEV)
    tok = torch.randint(0, 60000, (3, 2, 4), generator=g, device=DEV, dtype=torch.int32)
    u = torch.randint(0, 1 << 24, (2, 13), generator=g, device=DEV, dtype=torch.int32)
    sq.sq_spec_accept_multi(rows[:, :, :3].permute(2, 0, 1, 3).contiguous(), rows, tok, u, 1.0)  # 56 rows' scratch
    first = check(b, kd, v, temp, 500 + b)
    w, x = (torch.randn((n, 6400), generator=g, device=DEV).half() for n in (256, 100))
    _lib.sq_prefill_linear_f16(x, w, torch.empty((100, 256), device=DEV))  # partial sums of its K parts
    assert np.array_equal(first, check(b, kd, v, temp, 500 + b))
