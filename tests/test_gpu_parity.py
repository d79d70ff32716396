"""GPU parity: every HIP entry point against the CPU oracle on the same seeded
inputs, element by element.  Quantized codes, scales and accept decisions are
compared bit for bit; GEMV/GEMM outputs within max |y - y_ref| / sum |x w'|
<= 2e-3; softmax probabilities within 1e-5 absolute.  Shapes span several
tiles with ragged tails and include the degenerate cases."""
import numpy as np
import pytest
import torch
from scipy import special, stats

import oracle
import paper_2609_21704_amd as sq
from paper_2609_21704_amd import synth
from accept_compare import check_accept

pytestmark = pytest.mark.gpu
DEV = "cuda"
GEMV_TOL = 2e-3
PROB_TOL = 1e-5


def bits16(t: torch.Tensor) -> np.ndarray:
    return t.detach().cpu().contiguous().view(torch.int16).numpy().view(np.uint16)


def special_rows(w: torch.Tensor) -> torch.Tensor:
    """Overwrite the first rows with degenerate patterns (needs n >= 6)."""
    w = w.clone()
    n, k = w.shape
    if n >= 6:
        w[0] = 0.0                                             # all-zero row / groups
        w[1] = 0.0
        w[1, k // 3] = 1.0                                     # one-hot
        w[2] = torch.linspace(-1e-6, 1e-6, k).to(torch.float16)  # fp16 subnormals
        w[3] = -w[3].abs()                                     # all negative
        w[3, 0] = -0.0
        w[4] = w[4].abs()                                      # all positive
        w[5, : min(k, 64)] = 65504.0                           # fp16 extremes
        w[5, min(k, 64) // 2: min(k, 64)] = -65504.0
    return w


# ----------------------------------------------------------- quantizers ----
INT4_SHAPES = [(1, 128), (37, 384), (896, 896), (128, 896), (4864, 896), (896, 4864), (129, 3584)]


@pytest.mark.parametrize("n,k", INT4_SHAPES)
def test_quantize_int4_bit_exact(n, k):
    w = special_rows(synth.normal_f16((n, k), 0.02, synth.stream_seed(0, n, k)))
    codes, scales, zeros = sq.sq_quantize_int4_g128(w.to(DEV))
    c_ref, s_ref, z_ref = oracle.quantize_int4_g128(bits16(w))
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    assert np.array_equal(bits16(scales), s_ref)
    assert np.array_equal(bits16(zeros), z_ref)


def test_quantize_int4_nonfinite_flag():
    w = synth.normal_f16((4, 256), 0.02, 5)
    w[2, 200] = float("nan")
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    codes, scales, zeros = sq.sq_quantize_int4_g128(w.to(DEV), nonfinite_flag=flag)
    assert int(flag.item()) == 1
    assert bits16(scales)[2, 1] == 0x7E00 and np.all(codes.cpu().numpy()[2, 64:] == 0)
    ok = torch.zeros(1, dtype=torch.int32, device=DEV)
    sq.sq_quantize_int4_g128(synth.normal_f16((4, 256), 0.02, 6).to(DEV), nonfinite_flag=ok)
    assert int(ok.item()) == 0


FP8_SHAPES = [(1, 16), (37, 400), (896, 896), (128, 896), (4864, 896), (896, 4864), (5, 18944)]


@pytest.mark.parametrize("n,k", FP8_SHAPES)
def test_quantize_fp8_bit_exact(n, k):
    w = special_rows(synth.normal_f16((n, k), 0.02, synth.stream_seed(1, n, k)))
    codes, scales = sq.sq_quantize_fp8_e4m3(w.to(DEV))
    c_ref, s_ref = oracle.quantize_fp8_e4m3(bits16(w))
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))


def test_quantize_fp8_nonfinite_flag():
    w = synth.normal_f16((3, 64), 0.02, 7)
    w[1, 5] = float("inf")
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    codes, scales = sq.sq_quantize_fp8_e4m3(w.to(DEV), nonfinite_flag=flag)
    assert int(flag.item()) == 1
    assert np.isnan(scales.cpu().numpy()[1]) and np.all(codes.cpu().numpy()[1] == 0)


# every row-length range of the FP8 kernels at its edges, one cell past each, and the two-pass rows
@pytest.mark.parametrize("k", [16, 512, 1024, 1040, 2048, 2064, 3584, 3600, 4096, 4112, 8192, 8208, 16384, 16400,
                               32768, 32784])
def test_quantize_fp8_row_lengths(k):
    w = special_rows(synth.normal_f16((7, k), 0.02, synth.stream_seed(2, k)))
    codes, scales = sq.sq_quantize_fp8_e4m3(w.to(DEV))
    c_ref, s_ref = oracle.quantize_fp8_e4m3(bits16(w))
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))


def test_quantize_fp8_every_half():
    """All 63488 finite halves, by magnitude, in rows of 992: every rounding and tie under many row scales."""
    mags = np.arange(0x7C00, dtype=np.uint16)
    h = np.stack([mags, mags | 0x8000], -1).reshape(64, 992)
    w = torch.from_numpy(h.view(np.float16).copy())
    codes, scales = sq.sq_quantize_fp8_e4m3(w.to(DEV))
    c_ref, s_ref = oracle.quantize_fp8_e4m3(h)
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))


@pytest.mark.parametrize("unit", [1.0, 2.0 ** -14, 2.0 ** -24, 0.0371, 777.0])
def test_quantize_int4_ties(unit):
    """Groups of multiples of half a step (exact ties where the step is a half itself), ranges on either side of zero."""
    g = torch.Generator().manual_seed(3)
    steps = torch.randint(-30, 31, (61, 3 * 128), generator=g).double()
    steps[::3] = steps[::3].abs()
    steps[1::3] = -steps[1::3].abs()
    w = (steps * (0.5 * unit)).half() if unit != 2.0 ** -24 else (steps * unit).half()
    codes, scales, zeros = sq.sq_quantize_int4_g128(w.to(DEV))
    c_ref, s_ref, z_ref = oracle.quantize_int4_g128(bits16(w))
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    assert np.array_equal(bits16(scales), s_ref)
    assert np.array_equal(bits16(zeros), z_ref)


# ----------------------------------------------------------------- GEMV ----
# (3, 8192) and (2, 16384): a few rows with long rows, so tasks span several
# wavefronts of one workgroup with idle wavefronts between them
GEMV_SHAPES = [(1, 128), (37, 384), (896, 896), (4864, 896), (896, 4864), (257, 3584), (130, 18944), (3, 8192),
               (2, 16384)]


def _gemv_inputs(m, n, k, seed):
    w = synth.normal_f16((n, k), 0.02, synth.stream_seed(seed, 1, n, k))
    x = synth.normal_f16((m, k), 1.0, synth.stream_seed(seed, 2, m, k))
    return w, x


@pytest.mark.parametrize("n,k", GEMV_SHAPES)
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 8])
def test_qgemv_w4a16_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 10)
    wd, xd = w.to(DEV), x.to(DEV)
    codes, scales, zeros = sq.sq_quantize_int4_g128(wd)
    c_ref, s_ref, z_ref = oracle.quantize_int4_g128(bits16(w))
    y_ref, d_ref = oracle.qgemv_w4a16(bits16(x), c_ref, s_ref, z_ref)
    for dt in (torch.float32, torch.float16):
        y = sq.sq_qgemv_w4a16(xd, codes, scales, zeros, y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, (dt, err)


@pytest.mark.parametrize("n,k", [(1, 16), (37, 400), (896, 896), (4864, 896), (896, 4864), (257, 3584),
                                 (130, 18944), (3, 8192), (5, 4096)])
@pytest.mark.parametrize("m", [1, 2, 4, 5, 8])
def test_qgemv_w8a16_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 11)
    wd, xd = w.to(DEV), x.to(DEV)
    codes, scales = sq.sq_quantize_fp8_e4m3(wd)
    c_ref, s_ref = oracle.quantize_fp8_e4m3(bits16(w))
    y_ref, d_ref = oracle.qgemv_w8a16(bits16(x), c_ref, s_ref)
    for dt in (torch.float32, torch.float16):
        y = sq.sq_qgemv_w8a16(xd, codes, scales, y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, (dt, err)


# Few rows with long rows: each task's steps are split over a team of
# wavefronts, some of which take more steps than others.  W4 (4096 k per
# step): 3, 5, 6, 7 and 8 steps, then two 8-step K slices.  W8 (2048 k per
# step): 3, 10 and 15 steps.
TEAM_W4 = [(1, 37, 12288), (1, 37, 18944), (1, 37, 24576), (1, 37, 28672), (1, 37, 32768), (1, 5, 65536)]
TEAM_W8 = [(1, 37, 6144), (1, 37, 20480), (1, 37, 30720)]


@pytest.mark.parametrize("m,n,k", TEAM_W4)
def test_qgemv_w4a16_team_sizes(m, n, k):
    test_qgemv_w4a16_parity(m, n, k)


@pytest.mark.parametrize("m,n,k", TEAM_W8)
def test_qgemv_w8a16_team_sizes(m, n, k):
    test_qgemv_w8a16_parity(m, n, k)


# The row-block kernel (INT4, m <= 2): a workgroup per CU owns a block of
# rows and its wavefronts walk equal runs of the block's bytes, which start
# and end inside rows.  Blocks of 14 rows (the 7B down projection), of 3 or 4
# rows (1000 and 511 over the CUs), of one row (257), activations of up to
# 147 KB in LDS; rows of 2048 and 3584 k, where a step of 64 pieces meets
# three rows, with many rows per block; 5120 k with four-row tasks in the
# other kernel (the idle-lane rule picks this one).
LONG_W4 = [(1, 3584, 18944), (2, 1000, 4864), (1, 511, 9600), (2, 511, 9600), (1, 257, 65536), (2, 300, 32768),
           (1, 20000, 2048), (2, 9000, 3584), (1, 4608, 3584), (1, 40000, 5120)]


@pytest.mark.parametrize("m,n,k", LONG_W4)
def test_qgemv_w4a16_long_rows(m, n, k):
    test_qgemv_w4a16_parity(m, n, k)


# Short rows on the row-block kernel: 16 .. 30 pieces a row, so that a step of
# 64 pieces meets up to five rows (1024 .. 1280 k) or four (1408 .. 1920 k);
# ragged row counts, blocks of one row up to hundreds of rows.
SHORT_W4 = [(1, 4097, 1024), (2, 777, 1024), (1, 300, 1152), (2, 20011, 1280), (1, 2048, 1536), (2, 1536, 1536),
            (1, 151936, 1536), (1, 5003, 1408), (2, 257, 1920), (1, 33333, 1792)]


@pytest.mark.parametrize("m,n,k", SHORT_W4)
def test_qgemv_w4a16_short_rows(m, n, k):
    test_qgemv_w4a16_parity(m, n, k)


# So many row tiles per workgroup that up to 16 rows' chunk partial sums,
# 64 m bytes a tile, exceed their 40 KB of LDS even in one chunk a tile (over 256
# CUs 163840 weight rows at m = 16, 327680 at m = 8): the parent's projections
# take another kernel, the drafts' the padded two-tile form.  The smaller sizes fit.
@pytest.mark.parametrize("n,k", [(140000, 128), (170000, 256)])
def test_verify_gemm_many_tiles_m16(n, k):
    m = 16
    w = synth.normal_f16((n, k), 0.02, 51)
    x = synth.normal_f16((m, k), 1.0, 52)
    y_ref, d_ref = oracle.gemm_f16(bits16(x), bits16(w))
    y = sq.sq_verify_gemm_f16(x.to(DEV), w.to(DEV), y_dtype=torch.float32)
    assert oracle.normalised_error(y.cpu().numpy(), y_ref, d_ref) <= GEMV_TOL


@pytest.mark.parametrize("n", [300000, 340000])
def test_qgemv_w8a16_many_tiles_m8(n):
    m, k = 8, 256
    rng = np.random.default_rng(53)
    codes = rng.integers(0, 256, size=(n, k), dtype=np.uint8)
    codes[(codes & 0x7F) == 0x7F] = 0  # no NaN codes
    scales = rng.uniform(1e-4, 1e-3, size=n).astype(np.float32)
    x = synth.normal_f16((m, k), 1.0, 54)
    y_ref, d_ref = oracle.qgemv_w8a16(bits16(x), codes, scales)
    y = sq.sq_qgemv_w8a16(x.to(DEV), torch.from_numpy(codes).to(DEV), torch.from_numpy(scales).to(DEV),
                          y_dtype=torch.float32)
    assert oracle.normalised_error(y.cpu().numpy(), y_ref, d_ref) <= GEMV_TOL


@pytest.mark.parametrize("m,n", [(8, 340000), (5, 530000)])
def test_qgemv_w4a16_many_tiles(m, n):
    test_qgemv_w4a16_parity(m, n, 256)


def test_qgemv_w8a16_every_code_decodes_exactly():
    """Row c holds code c at column 0 (NaN codes replaced by 0); x = e_0."""
    n, k = 256, 32
    codes = np.zeros((n, k), np.uint8)
    codes[:, 0] = np.arange(256)
    codes[0x7F, 0] = codes[0xFF, 0] = 0
    scales = np.ones(n, np.float32)
    x = np.zeros((1, k), np.float16)
    x[0, 0] = 1.0
    y = sq.sq_qgemv_w8a16(torch.from_numpy(x).to(DEV), torch.from_numpy(codes).to(DEV),
                          torch.from_numpy(scales).to(DEV)).cpu().numpy()[0]
    y_ref, _ = oracle.qgemv_w8a16(x, codes, scales)
    assert np.array_equal(y.astype(np.float64), y_ref[0])


def test_qgemv_w4a16_closed_forms():
    k = 512
    x = synth.normal_f16((3, k), 1.0, 3)
    # identity: one-hot groups give 1.00067138671875 * x
    eye = torch.eye(k, dtype=torch.float16)
    codes, scales, zeros = sq.sq_quantize_int4_g128(eye.to(DEV))
    y = sq.sq_qgemv_w4a16(x.to(DEV), codes, scales, zeros).cpu().double().numpy()
    ref = 1.00067138671875 * x.double().numpy()
    d = np.abs(ref)
    assert np.max(np.abs(y - ref) / np.maximum(d, 1e-30)) <= GEMV_TOL
    # all-zero weights give exact zeros
    zc, zs, zz = sq.sq_quantize_int4_g128(torch.zeros((9, k), dtype=torch.float16, device=DEV))
    assert torch.count_nonzero(sq.sq_qgemv_w4a16(x.to(DEV), zc, zs, zz)).item() == 0


# ------------------------------------------------------------ verify GEMM ----
GEMM_SHAPES = [(1, 8), (37, 136), (896, 896), (4864, 896), (896, 4864), (100, 3584), (33, 18944)]


@pytest.mark.parametrize("n,k", GEMM_SHAPES)
@pytest.mark.parametrize("m", [1, 5, 7, 16, 17, 36, 48, 64])
def test_verify_gemm_f16_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 12)
    y_ref, d_ref = oracle.gemm_f16(bits16(x), bits16(w))
    for dt in (torch.float32, torch.float16):
        y = sq.sq_verify_gemm_f16(x.to(DEV), w.to(DEV), y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, (dt, err)


# The row-block verify kernel (m <= 8): the 7B q|k|v shape, activations of
# 8 x 8192 (two staging batches), rows of 768 k (a step meets three rows),
# 32768 rows of 512 k (the row limit), m = 7 at 5120 k, k % 16 == 8 (not
# whole pieces: another kernel takes it), and activations too large for one
# workgroup, where two workgroups share each row block, one per half of K
# (the 7B down projection among them).
ROWS_VERIFY = [(5, 4608, 3584), (8, 3000, 8192), (3, 1500, 768), (1, 32768, 512), (7, 5000, 5120),
               (5, 2000, 1032), (2, 33, 2048), (5, 1000, 18944), (8, 700, 12288), (5, 3584, 18944)]


@pytest.mark.parametrize("m,n,k", ROWS_VERIFY)
def test_verify_gemm_row_blocks(m, n, k):
    test_verify_gemm_f16_parity(m, n, k)


@pytest.mark.parametrize("m", [1, 5, 36])
def test_verify_gemm_identity_is_exact(m):
    k = 384
    x = synth.normal_f16((m, k), 1.0, 4)
    y = sq.sq_verify_gemm_f16(x.to(DEV), torch.eye(k, dtype=torch.float16, device=DEV))
    assert torch.equal(y.cpu(), x.float())


# --------------------------------------------------------------- accept ----
def _accept_case(b, kd, v, seed, temp, token_mode="sampled", sd=2.0, noise=0.5):
    """draft ~ N(0, sd), target = draft + N(0, noise) (bonus row fresh); tokens [kd][b] drawn from q."""
    draft = synth.normal_f32((kd, b, v), sd, synth.stream_seed(seed, 1))
    target = torch.empty((b, kd + 1, v), dtype=torch.float32)
    eps = synth.normal_f32((b, kd + 1, v), noise, synth.stream_seed(seed, 2))
    target[:, :kd] = draft.permute(1, 0, 2) + eps[:, :kd]
    target[:, kd] = synth.normal_f32((b, v), sd, synth.stream_seed(seed, 3))
    u24 = synth.uniform_u24((b, kd + 1), synth.stream_seed(seed, 4))
    if kd == 0:
        tok = torch.zeros((0, b), dtype=torch.int32)
    elif token_mode == "sampled" and temp > 0:
        q = oracle.softmax(draft.reshape(kd * b, v).numpy(), float(np.float32(temp))).reshape(kd, b, v)
        r = np.random.default_rng(seed).random((kd, b))
        tok = np.minimum((r[..., None] >= np.cumsum(q, axis=2)).sum(axis=2), v - 1).astype(np.int32)  # [kd][b]
        tok = torch.from_numpy(np.ascontiguousarray(tok))
    else:
        tok = synth.tokens((kd, b), v, synth.stream_seed(seed, 5))
    return draft, target, tok, u24


def _run_accept(draft, target, tok, u24, temp, want_pq=False):
    b, kd1, v = target.shape
    kd = kd1 - 1
    q_out = torch.empty((kd, b, v), dtype=torch.float32, device=DEV) if want_pq and kd > 0 else None
    p_out = torch.empty((b, kd1, v), dtype=torch.float32, device=DEV) if want_pq else None
    n, t = sq.sq_spec_accept(draft.to(DEV) if kd > 0 else None, target.to(DEV), tok.to(DEV) if kd > 0 else None,
                             u24.to(DEV), temp, q_out=q_out, p_out=p_out)
    return n.cpu().numpy(), t.cpu().numpy(), q_out, p_out


ACCEPT_CASES = [
    (1, 4, 4096, 1.0), (1, 4, 151936, 1.0), (4, 8, 151936, 1.0), (3, 0, 1000, 1.0), (7, 3, 8, 0.7),
    (2, 64, 300, 1.0), (64, 2, 5000, 1.3), (16, 6, 152064, 1.0), (5, 1, 4097, 0.5),
    # 256 chunk partials per row held in registers, then one more read from memory
    (2, 3, 262144, 1.0), (2, 3, 262145, 1.0),
]


@pytest.mark.parametrize("b,kd,v,temp", ACCEPT_CASES)
@pytest.mark.parametrize("token_mode", ["sampled", "uniform"])
def test_spec_accept_parity(b, kd, v, temp, token_mode):
    """Decisions and draws bit-exact against the oracle run on the kernel's
    own fp32 distributions; end to end against the oracle's own softmax up to
    counted near-ties; the same bits without q_out / p_out."""
    temp = float(np.float32(temp))
    draft, target, tok, u24 = _accept_case(b, kd, v, 100 + b + kd, temp, token_mode)
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, temp, want_pq=True)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), temp, n, t,
                 q_out.cpu().numpy() if q_out is not None else None, p_out.cpu().numpy())
    n2, t2, _, _ = _run_accept(draft, target, tok, u24, temp)
    assert np.array_equal(n, n2) and np.array_equal(t, t2)


def test_spec_accept_zero_residual_falls_back_to_p_n():
    """Rejections that leave no residual mass on the 2^-60 grid: a drafted
    token outside [0, v) or masked in both rows (p(x) = q(x) = 0), with the
    parent's row equal to the draft's row, so max(0, p - q) = 0 everywhere and
    the token is drawn from p_n.  Other sequences keep the ordinary path."""
    b, kd, v = 12, 4, 9000
    draft, target, tok, u24 = _accept_case(b, kd, v, 61, 1.0, "uniform")
    for s in range(b):
        i = s % kd
        target[s, i] = draft[i, s]
        if s % 3 == 0:
            tok[i, s] = -1 if s % 2 else v
        elif s % 3 == 1:
            draft[i, s, 17] = -np.inf
            target[s, i, 17] = -np.inf
            tok[i, s] = 17
        # s % 3 == 2: an ordinary sequence whose row i happens to equal the draft
        for j in range(i):
            target[s, j] = draft[j, s]          # earlier positions: p = q, always accepted
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, 1.0, want_pq=True)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), 1.0, n, t,
                 q_out.cpu().numpy(), p_out.cpu().numpy())
    for s in range(b):
        if s % 3 != 2:
            assert n[s] == s % kd
            assert 0 <= t[s] < v and np.isfinite(target[s, n[s], t[s]].item())


def test_spec_accept_masked_chunks():
    """-inf logits over whole chunks (1024 logits each) and scattered tokens: masked
    tokens get probability 0 and are never emitted; rows of masked chunks
    merge like the oracle's softmax."""
    b, kd, v = 6, 3, 20000
    draft, target, tok, u24 = _accept_case(b, kd, v, 67, 1.0, "uniform")
    target[0, 0, 4096:8192] = -np.inf        # one whole chunk
    target[1, :, :12288] = -np.inf           # three whole chunks of every target row
    draft[:, 2, 8192:] = -np.inf             # every chunk but the first two of the draft rows
    target[3, 1, ::3] = -np.inf              # scattered
    draft[2, 4, 12288:16384] = -np.inf
    target[5, 3, :19999] = -np.inf           # a bonus row with one finite logit
    tok[0, 1] = 5                            # masked in the parent: always rejected
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, 1.0, want_pq=True)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), 1.0, n, t,
                 q_out.cpu().numpy(), p_out.cpu().numpy())
    _, _, q_ref, p_ref = oracle.spec_accept(draft.numpy(), target.numpy(), tok.numpy(),
                                            u24.numpy().view(np.uint32), 1.0, want_pq=True)
    assert np.max(np.abs(p_out.cpu().numpy() - p_ref)) <= PROB_TOL
    assert np.max(np.abs(q_out.cpu().numpy() - q_ref)) <= PROB_TOL
    assert np.all(p_out.cpu().numpy()[np.isinf(target.numpy())] == 0)
    assert n[1] == 0 and all(np.isfinite(target[s, n[s], t[s]].item()) for s in range(b))


@pytest.mark.parametrize("temp", [1.0, 0.0])
def test_spec_accept_rows_without_a_distribution(temp):
    """A NaN or +inf logit, or a row with no finite logit, makes its sequence
    return n_accepted = next_token = -1 (NaN rows in p_out / q_out); the other
    sequences are unaffected."""
    b, kd, v = 8, 2, 5000
    draft, target, tok, u24 = _accept_case(b, kd, v, 71, 1.0, "uniform")
    target[1, 2, 4500] = float("nan")
    target[2, 0, 7] = float("inf")
    target[3, 1, :] = -np.inf
    draft[1, 4, 100] = float("nan")          # draft rows matter only at T > 0
    draft[0, 5, :] = -np.inf
    target[6, 0, :4096] = -np.inf            # a masked chunk only: valid
    want = temp > 0
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, temp, want_pq=want)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), temp, n, t,
                 q_out.cpu().numpy() if want else None, p_out.cpu().numpy() if want else None)
    bad = [1, 2, 3, 4, 5] if temp > 0 else [1, 2, 3]
    assert all(n[s] == -1 and t[s] == -1 for s in bad)
    assert all(n[s] >= 0 and t[s] >= 0 for s in range(b) if s not in bad)
    if want:
        assert np.all(np.isnan(p_out[1, 2].cpu().numpy())) and np.all(np.isnan(q_out[1, 4].cpu().numpy()))
        assert not np.any(np.isnan(p_out[6].cpu().numpy()))


@pytest.mark.parametrize("b,kd,v,temp", [(1, 4, 4096, 1.0), (4, 8, 151936, 1.0), (3, 0, 1000, 0.8)])
def test_spec_accept_probabilities(b, kd, v, temp):
    temp = float(np.float32(temp))
    draft, target, tok, u24 = _accept_case(b, kd, v, 7, temp)
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, temp, want_pq=True)
    n_ref, t_ref, q_ref, p_ref = oracle.spec_accept(draft.numpy(), target.numpy(), tok.numpy(),
                                                    u24.numpy().view(np.uint32), temp, want_pq=True)
    assert np.max(np.abs(p_out.cpu().numpy() - p_ref)) <= PROB_TOL
    if kd > 0:
        assert np.max(np.abs(q_out.cpu().numpy() - q_ref)) <= PROB_TOL
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), temp, n, t,
                 q_out.cpu().numpy() if kd > 0 else None, p_out.cpu().numpy())


@pytest.mark.parametrize("b,kd,v", [(5, 4, 4096), (3, 0, 100), (200, 3, 50), (2, 8, 151936)])
def test_spec_accept_greedy(b, kd, v):
    draft, target, tok, u24 = _accept_case(b, kd, v, 9, 0.0, "uniform")
    target[0, 0] = 1.0                               # ties -> smallest index
    am = target.argmax(dim=2).to(torch.int32)
    if kd > 0:
        tok = am[:, :kd].t().contiguous()
        tok[kd // 2, 1 % b] = (tok[kd // 2, 1 % b] + 1) % v
    n, t, _, _ = _run_accept(draft, target, tok, u24, 0.0)
    n_ref, t_ref, _, _ = oracle.spec_accept(draft.numpy(), target.numpy(), tok.numpy(), None, 0.0)
    assert np.array_equal(n, n_ref) and np.array_equal(t, t_ref)


@pytest.mark.parametrize("temp,kd,v", [(0.0, 0, 1), (0.0, 2, 4097), (1.0, 0, 1025)])
def test_spec_accept_more_sequences_than_arrival_slots(temp, kd, v):
    """Sequences past the first 65536 rows (or sequences) of a call get what they get in a call of their own."""
    b, tail = 65536 // (kd + 1) + 40, 60
    g = torch.Generator(device=DEV).manual_seed(v)
    target = torch.randn((b, kd + 1, v), generator=g, device=DEV)
    draft = torch.randn((kd, b, v), generator=g, device=DEV) if kd else None
    tok = target[:, :kd].argmax(-1).t().to(torch.int32).contiguous() if kd else None
    if kd:
        tok[1, ::3] = (tok[1, ::3] + 1) % v
    u = torch.randint(0, 1 << 24, (b, kd + 1), generator=g, device=DEV, dtype=torch.int32)
    n, t = sq.sq_spec_accept(draft, target, tok, u, temp)
    n2, t2 = sq.sq_spec_accept(draft[:, -tail:].contiguous() if kd else None, target[-tail:].contiguous(),
                               tok[:, -tail:].contiguous() if kd else None, u[-tail:].contiguous(), temp)
    assert torch.equal(n[-tail:], n2) and torch.equal(t[-tail:], t2) and int(t.min()) >= 0
    if temp == 0.0:
        assert torch.equal(t, target[torch.arange(b, device=DEV), n.long()].argmax(-1).to(torch.int32))


def test_spec_accept_edge_tokens_and_equal_distributions():
    b, kd, v = 6, 4, 333
    draft, target, tok, u24 = _accept_case(b, kd, v, 21, 1.0, "uniform")
    tok[0, 0] = -1          # [position][sequence]
    tok[2, 1] = v
    tok[1, 2] = 1 << 30
    target[3, :kd] = draft[:, 3]                     # p = q for sequence 3: all accepted
    u24[4] = (1 << 24) - 1
    u24[5] = 0
    n, t, q_out, p_out = _run_accept(draft, target, tok, u24, 1.0, want_pq=True)
    check_accept(draft.numpy(), target.numpy(), tok.numpy(), u24.numpy(), 1.0, n, t,
                 q_out.cpu().numpy(), p_out.cpu().numpy())
    assert n[0] == 0 and n[3] == kd


def test_spec_accept_chi_square_on_gpu():
    """10^6 sequences at V = 8, kd = 4: acceptance law and per-position token law."""
    rng = np.random.default_rng(3)
    b, kd, v = 1_000_000, 4, 8
    dl = rng.normal(0, 1.2, (kd, v)).astype(np.float32)
    tl = np.concatenate([dl + rng.normal(0, 0.8, (kd, v)).astype(np.float32),
                         rng.normal(0, 1, (1, v)).astype(np.float32)])
    q = special.softmax(dl.astype(np.float64), axis=1)
    p = special.softmax(tl.astype(np.float64), axis=1)
    x = np.minimum((rng.random((b, kd))[..., None] >= np.cumsum(q, axis=1)[None]).sum(axis=2), v - 1).astype(np.int32)
    u24 = rng.integers(0, 1 << 24, (b, kd + 1)).astype(np.int32)
    draft = torch.from_numpy(np.ascontiguousarray(np.broadcast_to(dl[:, None, :], (kd, b, v))))
    target = torch.from_numpy(np.ascontiguousarray(np.broadcast_to(tl[None], (b, kd + 1, v))))
    n, nxt, _, _ = _run_accept(draft, target, torch.from_numpy(np.ascontiguousarray(x.T)), torch.from_numpy(u24), 1.0)
    crit = lambda dof: stats.chi2.ppf(1 - 1e-3, dof)
    beta = np.minimum(p[:kd], q).sum(axis=1)
    law = np.array([np.prod(beta[:i]) * (1 - beta[i]) for i in range(kd)] + [np.prod(beta)])
    obs = np.bincount(n, minlength=kd + 1)
    assert np.sum((obs - b * law) ** 2 / (b * law)) < crit(kd)
    for i in range(kd + 1):
        reached = n >= i
        tok = np.where(n[reached] > i, x[reached, min(i, kd - 1)], nxt[reached])
        cnt = np.bincount(tok, minlength=v)
        exp = reached.sum() * p[i]
        assert np.sum((cnt - exp) ** 2 / exp) < crit(v - 1), i


# ---------------------------------------------------------- determinism ----
def test_repeat_runs_are_bitwise_identical():
    w, x = _gemv_inputs(5, 4864, 896, 13)
    wd, xd = w.to(DEV), x.to(DEV)
    c4 = sq.sq_quantize_int4_g128(wd)
    c8 = sq.sq_quantize_fp8_e4m3(wd)
    outs = []
    for _ in range(2):
        outs.append((sq.sq_qgemv_w4a16(xd[:1], *c4), sq.sq_qgemv_w8a16(xd[:4], *c8), sq.sq_verify_gemm_f16(xd, wd)))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    draft, target, tok, u24 = _accept_case(4, 8, 151936, 5, 1.0)
    r1 = _run_accept(draft, target, tok, u24, 1.0)
    r2 = _run_accept(draft, target, tok, u24, 1.0)
    assert np.array_equal(r1[0], r2[0]) and np.array_equal(r1[1], r2[1])


# ------------------------------------------- large matrices (matrix cores) ----
# Matrices of 64 MB and more stream through the matrix-core kernel: ragged
# row counts and k (partial 16-byte slabs), and k long enough that the
# activations are cut into slices summed by a second kernel.
# the last three: K cut into two slices that meet per output value, and into nine
LARGE_GEMM = [(1, 16384, 4096), (5, 16384, 4096), (16, 16384, 4096), (5, 16381, 4104), (7, 16381, 4104),
              (5, 2048, 18944), (3, 1100, 40000), (16, 2048, 32768)]


@pytest.mark.parametrize("m,n,k", LARGE_GEMM)
def test_verify_gemm_f16_large_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 14)
    y_ref, d_ref = oracle.gemm_f16(bits16(x), bits16(w))
    wd, xd = w.to(DEV), x.to(DEV)
    for dt in (torch.float32, torch.float16):
        y = sq.sq_verify_gemm_f16(xd, wd, y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, (dt, err)
    assert torch.equal(sq.sq_verify_gemm_f16(xd, wd), sq.sq_verify_gemm_f16(xd, wd))


# m = 17..64 on the matrix-core streaming kernel (several 16-row activation
# tiles): chunks of a task spread over the wavefronts with their partial sums
# in LDS (m = 17: two K slices meeting per value; m = 36 at 4104 k: a partial
# slab and three slices added by the second kernel), and the direct mode,
# where the partial sums would not fit (whole tasks per wavefront: one slice
# at m = 20, several slices at m = 48, 64 and 33), over ragged row counts
WIDE_GEMM = [(17, 16384, 4096), (36, 16381, 4104), (20, 151936, 1024), (48, 37888, 3584), (64, 9001, 5120),
             (33, 2000, 18944)]


@pytest.mark.parametrize("m,n,k", WIDE_GEMM)
def test_verify_gemm_f16_wide_parity(m, n, k):
    test_verify_gemm_f16_large_parity(m, n, k)


# the last two: K cut into two slices
LARGE_W8 = [(1, 16384, 4096), (4, 16384, 4096), (8, 16384, 4096), (4, 16381, 4112), (8, 4096, 16384),
            (6, 4097, 16400)]


@pytest.mark.parametrize("m,n,k", LARGE_W8)
def test_qgemv_w8a16_large_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 15)
    wd, xd = w.to(DEV), x.to(DEV)
    codes, scales = sq.sq_quantize_fp8_e4m3(wd)
    c_ref, s_ref = oracle.quantize_fp8_e4m3(bits16(w))
    assert np.array_equal(codes.cpu().numpy(), c_ref)
    y_ref, d_ref = oracle.qgemv_w8a16(bits16(x), c_ref, s_ref)
    for dt in (torch.float32, torch.float16):
        y = sq.sq_qgemv_w8a16(xd, codes, scales, y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, (dt, err)
    assert torch.equal(sq.sq_qgemv_w8a16(xd, codes, scales), sq.sq_qgemv_w8a16(xd, codes, scales))


# ------------------------------------------ draft projections over many rows
# Above m = 8 the quantized copies run on the matrix cores (activation tiles
# of 16 rows): one, two, three and four tiles; K cut into slices (k = 18944 at
# m = 64); and a matrix with too many tiles per workgroup for the chunk
# partial sums at m = 16 (163840 rows and more over 256 CUs), which takes whole
# tasks per wavefront instead.
MANY_ROWS = [(9, 37, 384), (16, 896, 896), (17, 4864, 896), (33, 896, 4864), (48, 257, 3584), (64, 130, 3584),
             (64, 1024, 18944), (16, 140000, 256), (16, 170000, 256), (12, 4608, 3584)]


@pytest.mark.parametrize("m,n,k", MANY_ROWS)
def test_qgemv_many_rows_parity(m, n, k):
    w, x = _gemv_inputs(m, n, k, 16)
    wd, xd = w.to(DEV), x.to(DEV)
    codes, scales, zeros = sq.sq_quantize_int4_g128(wd)
    c_ref, s_ref, z_ref = oracle.quantize_int4_g128(bits16(w))
    y_ref, d_ref = oracle.qgemv_w4a16(bits16(x), c_ref, s_ref, z_ref)
    c8, s8 = sq.sq_quantize_fp8_e4m3(wd)
    c8_ref, s8_ref = oracle.quantize_fp8_e4m3(bits16(w))
    y8_ref, d8_ref = oracle.qgemv_w8a16(bits16(x), c8_ref, s8_ref)
    for dt in (torch.float32, torch.float16):
        y = sq.sq_qgemv_w4a16(xd, codes, scales, zeros, y_dtype=dt)
        err = oracle.normalised_error(y.float().cpu().numpy(), y_ref, d_ref)
        assert err <= GEMV_TOL, ("int4", dt, err)
        y8 = sq.sq_qgemv_w8a16(xd, c8, s8, y_dtype=dt)
        err = oracle.normalised_error(y8.float().cpu().numpy(), y8_ref, d8_ref)
        assert err <= GEMV_TOL, ("fp8", dt, err)
    # deterministic, and each row of the block is the single-row product of its row
    y1 = sq.sq_qgemv_w4a16(xd, codes, scales, zeros)
    assert torch.equal(y1, sq.sq_qgemv_w4a16(xd, codes, scales, zeros))
    row = sq.sq_qgemv_w4a16(xd[m - 1:m].contiguous(), codes, scales, zeros).cpu().numpy()[0]
    err = oracle.normalised_error(row, y_ref[m - 1], d_ref[m - 1])
    assert err <= GEMV_TOL
