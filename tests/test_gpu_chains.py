"""The accept call over several chains where its launches change: nodes whose later candidates the walk takes itself, or
only some of them, rows on both sides of the rule, and scratch with another call's tests and masses; against the oracle's
rule on the kernel's own fp32 distributions, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_21704_amd as sq
from test_gpu_multi import make_case

pytestmark = pytest.mark.gpu
DEV = "cuda"


def check(dl, tl, tok, u, temp):
    kd, b, c, v = dl.shape
    args = [a.to(DEV) for a in (dl, tl, tok, u)]
    q_out, p_out = torch.empty((kd, b, c, v), device=DEV), torch.empty((b, c, kd + 1, v), device=DEV)
    n, t, ch = [a.cpu().numpy() for a in sq.sq_spec_accept_multi(*args, temp, q_out=q_out, p_out=p_out)]
    again = [a.cpu().numpy() for a in sq.sq_spec_accept_multi(*args, temp)]
    assert all(np.array_equal(x, y) for x, y in zip((n, t, ch), again))
    want = oracle.multi_accept_probs(p_out.cpu().numpy(), q_out.cpu().numpy(), tok.numpy(), u.numpy().view(np.uint32))
    assert all(np.array_equal(x, y) for x, y in zip((n, t, ch), want)), ((n, t, ch), want)
    return n


# chains x logits: all later candidates in the walk (v < 4096); all by launches, one more chain and one less logit than
# that; some of them; the largest row of the walk and one more logit
@pytest.mark.parametrize("b,c,kd,v", [(4, 3, 2, 4095), (4, 3, 2, 4096), (3, 4, 2, 4096), (6, 6, 3, 8191), (3, 33, 1, 5000),
                                      (2, 20, 1, 32768), (2, 20, 1, 32769), (5, 8, 2, 1), (5, 8, 3, 40)])
@pytest.mark.parametrize("noise", [0.0, 12.0])
def test_chains_candidates_by_launches_and_by_the_walk(b, c, kd, v, noise):
    """Everything accepted early, then (into the scratch that left) next to nothing."""
    temp = 1.0 if c % 2 else 0.8
    n = check(*make_case(b, c, kd, v, seed=b * 100 + c, share=0.3, noise=noise), temp)
    if v > 1000:
        assert (n == kd).any() if noise == 0.0 else (n < kd).any()


@pytest.mark.parametrize("v", [900, 20000])
def test_chains_late_candidates_without_residual_mass(v):
    """Candidates that no row holds, more than the launches take: with p = q each one's rejection leaves no mass and the
    walk goes back to p; where the rows differ, the mass of the ones before counts."""
    b, c, kd = 5, 12, 2
    dl, tl, tok, u = make_case(b, c, kd, v, seed=3, share=0.0, noise=0.0)
    tok[0, 0] = v                                # no candidate of the root is in the row
    tok[0, 1, :10] = -1                          # the last two are
    tok[0, 2] = torch.arange(c, dtype=torch.int32)
    dl[0, 2, :, :c] = -np.inf                    # q = 0 there: never accepted at the first place
    tl[3, :, 0] += torch.randn(tl[3, :, 0].shape)
    tok[0, 3, :9] = -7
    n = check(dl, tl, tok, u, 1.0)
    assert n[0] == 0
