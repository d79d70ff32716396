"""Host-side validation of the prefill calls (no GPU: nothing is enqueued on an error)."""
import paper_2609_21704_amd as sq

A = 0x7F0000000000
B, C, D, E = (A + (i << 36) for i in range(1, 5))
NULL, SHAPE, ALIGN, ALIAS, NONFINITE, UNSUPPORTED = 1, 2, 3, 4, 5, 6


def test_prefill_linear_validation():
    lib = sq.load()
    f = lib.sq_prefill_linear_f16
    assert f(None, 4, 64, B, 8, C, 0, None) == NULL and f(A, 4, 64, B, 8, None, 0, None) == NULL
    for m, k, n in ((0, 64, 8), ((1 << 20) + 1, 64, 8), (4, 96, 8), (4, 0, 8), (4, 64, 0), (4, 1 << 20, 1 << 11)):
        assert f(A, m, k, B, n, C, 0, None) == SHAPE, (m, k, n)
    assert f(A, 4, 64, B, 7, C, 2, None) == SHAPE and f(A, 4, 64, B, 8, C, 3, None) == UNSUPPORTED
    assert f(A + 8, 4, 64, B, 8, C, 0, None) == ALIGN and f(A, 4, 64, B, 8, C + 4, 0, None) == ALIGN
    assert f(A, 4, 64, B, 8, A + 16, 0, None) == ALIAS
    g = lib.sq_prefill_linear_w4
    assert g(A, 4, 128, B, C, None, 8, D, 0, None) == NULL and g(A, 4, 192, B, C, D, 8, E, 0, None) == SHAPE
    assert g(A, 4, 128, B, C + 1, D, 8, E, 0, None) == ALIGN and g(A, 4, 128, B, C, D, 8, D, 0, None) == ALIAS
    h = lib.sq_prefill_linear_w8
    assert h(A, 4, 64, B, None, 8, D, 0, None) == NULL and h(A, 4, 64, B, C + 2, 8, D, 0, None) == ALIGN


def test_prefill_block_validation():
    lib = sq.load()

    def rope(rows=100, lb=128, cap=128, theta=1e6, q=C):
        return lib.sq_prefill_rope_kv_f16(A, None, 1, rows, 2, 1, B, 0, lb, cap, theta, q, D, E, None, None)

    assert rope(q=None) == NULL and rope(rows=129) == SHAPE and rope(cap=100) == SHAPE
    assert rope(theta=float("nan")) == NONFINITE and rope(theta=1.0) == SHAPE and rope(q=A + 16) == ALIAS

    def attn(rows=100, hq=2, out=E):
        return lib.sq_prefill_attention_f16(A, B, C, 1, rows, hq, 2, D, 0, 128, 128, out, None)

    assert attn(out=None) == NULL and attn(rows=129) == SHAPE and attn(hq=3) == SHAPE and attn(out=E + 8) == ALIGN
