"""Each attention kernel on its own: 256 and 128 queries per workgroup (attn_fwd<8> and <4>) and the key split
over 32 queries (attn_split), for every score format and probability path, at key tile counts that take the
prologue, the body of the four-way unrolled loop, each of its remainders, the tail iterations and several
batches of block means, with ragged last tiles down to one key. The number of heads chooses the kernel, and
the plan is asked which one it is, so a test cannot move to another kernel unnoticed.

Codes against the CPU oracle as in test_gpu_codes.py (INT8 with ExpCast bit for bit, hardware exponentials and
MXFP4 within a step, FP8 within the window of its product's error bound), outputs against its 64-bit sums,
the dumping variant against vc_attn_forward bit for bit. A call's heads repeat three inputs, and all
repetitions have to agree bit for bit (a missing wait would show as one that does not)."""
import numpy as np
import pytest

import oracle
import synthetic as S
from plans import forward_plan
from test_gpu_codes import UNSET, assert_codes_equal, f8_expcast_window, running_max_ends
from test_gpu_fp8qk import check_output_f8, flip_bound
from test_gpu_mx import rand_qkv
from test_gpu_parity import check_output, dev16, dev32

torch = pytest.importorskip("torch")
vc = pytest.importorskip("paper_2609_15810_amd")

pytestmark = pytest.mark.gpu
FORMATS = {"int8": vc.QK_INT8, "fp8": vc.QK_FP8, "mxfp4": vc.QK_MXFP4}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vc.lib()


def heads_for(queries, N, fmt="int8", p_mode=0, full=False, least=2):
    """The smallest number of heads with which the kernel of that many queries takes all rows (full: the rest
    behind full rounds of the 256-query kernel)."""
    for H in range(least, 700):
        n8, _, n4, _, n1 = forward_plan(N, H, FORMATS[fmt], p_mode)
        if ({256} if n8 else set()) | ({128} if n4 else set()) | ({32} if n1 else set()) == ({256, queries} if full else {queries}):
            return H
    raise AssertionError(f"no number of heads takes {N} tokens to the {queries}-query kernel")


def run(src, H, grid, fmt="int8", perm=None, q_perm=None, **opt):
    """(codes [H, N, 128 T], output [H, N, 128], both of the dumping variant) of H heads that repeat the ones in
    src = (Q, K, V); the output of vc_attn_forward has to be the same."""
    N = src[0].shape[2]
    T = -(-N // 128)
    pick = torch.arange(H) % src[0].shape[1]
    q, k, v = (dev16(x)[:, pick].contiguous() for x in src)
    perm, q_perm = (None if p is None else dev32(p)[:, pick].contiguous() for p in (perm, q_perm))
    A = vc.Attention(1, H, grid, vc.make_opts(qk_fmt=FORMATS[fmt], **opt), vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.prep(q, k, v, perm=perm, q_perm=q_perm)
    codes = torch.full((1, H, N, 128 * T), UNSET, dtype=torch.uint8, device="cuda")
    O1 = torch.full((1, H, N, 128), 0x7fc0, dtype=torch.int16, device="cuda")   # NaN: a row left out shows
    O2 = O1.clone()
    A.forward_codes(O1, codes, q_perm=q_perm)
    A.forward(O2, q_perm=q_perm)
    torch.cuda.synchronize()
    assert torch.equal(O1, O2), "the dumping variant changed the output"
    return codes[0], O1[0]


def repeats_agree(x, n):
    return all(torch.equal(x[h], x[h % n]) for h in range(n, x.shape[0]))


def values(o, n):
    return S.bits_to_f32(o[:n].cpu().numpy().view(np.uint16)).astype(np.float64)


def reached(queries, N):
    return queries != 32 or N > 256   # no key split up to two tiles


EVERY = [(q, N) for q in (256, 128, 32)
         for N in (100, 129, 300, 385, 513, 700, 833, 1000, 1100, 1400, 2500) if reached(q, N)]   # 1..9, 11, 20 tiles


@pytest.mark.parametrize("queries,N", EVERY)
def test_expcast_int8_codes(queries, N):
    n, grid = 2, (1, 1, N)
    src = rand_qkv(1, n, N, 7000 + N)
    perm, qp = S.random_perm(N, N, 1, n), S.random_perm(N, N + 1, 1, n)
    g, o = run(src, heads_for(queries, N), grid, perm=perm, q_perm=qp)
    pp = oracle.prep(*src, grid, perm=perm, q_perm=qp)
    rows = np.unique(np.concatenate([np.arange(0, N, 1 if N <= 700 else 5), [N - 1]])).astype(np.int32)
    assert_codes_equal(g[:n].cpu().numpy(), oracle.attention_codes(pp, rows), rows, f"{queries} N={N}")
    o_rows = np.stack([values(o, n)[h, qp[0, h, rows]] for h in range(n)])   # row i goes to token q_perm[i]
    check_output(o_rows, oracle.attention(pp, rows), f"{queries} N={N}")
    assert repeats_agree(g, n) and repeats_agree(o, n)


@pytest.mark.parametrize("fmt,p_mode", [("int8", 1), ("fp8", 0), ("fp8", 1), ("mxfp4", 0), ("mxfp4", 1)])
@pytest.mark.parametrize("queries,N", [(q, N) for q in (256, 128, 32) for N in (200, 300, 500, 513, 700, 833, 1500) if reached(q, N)])
def test_formats_and_paths(queries, N, fmt, p_mode):
    n, grid = 2, (1, 1, N)
    src = rand_qkv(1, n, N, 8000 + N)
    g, o = run(src, heads_for(queries, N, fmt, p_mode), grid, fmt, p_mode=p_mode)
    assert repeats_agree(g, n) and repeats_agree(o, n)
    pp = oracle.prep(*src, grid, qk_fmt={"int8": oracle.QK_INT8, "fp8": oracle.QK_FP8, "mxfp4": oracle.QK_MXFP4}[fmt])
    rows = np.unique(np.concatenate([np.arange(0, N, 37), [N - 1]])).astype(np.int32)
    sel = g[:n].cpu().numpy()[:, rows].astype(int)
    c = oracle.attention_codes(pp, rows, p_mode=p_mode).astype(int)
    ref, got = oracle.attention(pp, rows, p_mode=p_mode), values(o, n)[:, rows]
    if fmt == "fp8":
        for h in range(n):
            check_output_f8(got[h], ref[h], flip_bound(pp, h, rows, p_mode=p_mode), f"{queries} N={N} {fmt} {p_mode}")
            if p_mode == 0:
                lo, hi = f8_expcast_window(pp, h, rows)
                assert ((sel[h] >= lo) & (sel[h] <= hi)).all()
    else:
        assert np.abs(sel - c).max() <= 1 and (sel != c).mean() <= 1e-2
        check_output(got, ref, f"{queries} N={N} {fmt} {p_mode}")


@pytest.mark.parametrize("sigma,beta", [(40.0, 0.0), (200.0, -0.35)])
@pytest.mark.parametrize("queries", [256, 128, 32])
def test_huge_scores(queries, sigma, beta):
    """Running maxima between 2^16 and 2^27: the bytewise clip of each kernel's codes."""
    N, n = 1100, 2   # nine tiles: the steady loop, its remainder and the tail
    rng = np.random.default_rng(int(sigma))
    src = [S.bf16_bits((rng.standard_normal((1, n, N, 128)) * s).astype(np.float32)) for s in (sigma, sigma, 1.0)]
    g, o = run(src, heads_for(queries, N), (1, 1, N), sm_scale=1.0, beta=beta)
    pp = oracle.prep(*src, (1, 1, N))
    rows = np.arange(0, N, 3)
    ext = np.maximum(*(np.abs(x) for x in running_max_ends(pp, 0, rows, 1.0)))
    assert 2.0 ** 16 <= ext.max() < 2.0 ** 27
    assert_codes_equal(g[:n].cpu().numpy(), oracle.attention_codes(pp, rows, sm_scale=1.0, beta=beta), rows, f"{queries} {sigma}")
    check_output(values(o, n)[:, rows], oracle.attention(pp, rows, sm_scale=1.0, beta=beta), f"{queries} {sigma}")
    assert repeats_agree(g, n) and repeats_agree(o, n)


@pytest.mark.parametrize("queries", [256, 128, 32])
def test_domain(queries):
    """Rows are NaN where the running maximum after the first or the last tile reaches 2^27, and only there. Keys of
    equal channels, by head: the first tile's all beyond the limit; only those of one half of a wave's lanes; only
    those of the other half; the last tile's beyond the limit upwards."""
    N = 700
    far = 1000.0   # with queries of 1000 in all channels: 1.3e8 in logits, 1.8e8 in log2 units
    i = np.arange(N)
    half = (i >> 2) & 1
    k = np.stack([np.where(i < 128, -far, 0.0), np.where((i < 128) & (half == 0), -far, 0.0),
                  np.where((i < 128) & (half == 1), -far, 0.0), np.where(i >= 640, far, 0.0)])
    n = len(k)
    Q = S.bf16_bits(np.full((1, n, N, 128), far, np.float32))
    K = S.bf16_bits(np.broadcast_to(k[None, :, :, None], (1, n, N, 128)).astype(np.float32))
    V = S.bf16_bits(np.random.default_rng(3).standard_normal((1, n, N, 128)).astype(np.float32))
    opt = dict(rope=False, hadamard=False, smooth_k=False)
    g, o = run((Q, K, V), heads_for(queries, N, least=n), (1, 1, N), sm_scale=1.0, **opt)
    v = values(o, n)
    assert np.isnan(v[0]).all() and np.isnan(v[3]).all()
    pp = oracle.prep(Q, K, V, (1, 1, N), **opt)
    rows = np.arange(0, N, 3)
    assert_codes_equal(g[1:3].cpu().numpy(), oracle.attention_codes(pp, rows, bh=[1, 2], sm_scale=1.0), rows, f"{queries}")
    check_output(v[1:3][:, rows], oracle.attention(pp, rows, bh=[1, 2], sm_scale=1.0), f"{queries}")
    assert repeats_agree(g, n) and repeats_agree(o, n)


@pytest.mark.parametrize("queries,N", [(128, 1500), (32, 1500), (32, 1000)])
def test_full_rounds_and_a_rest(queries, N):
    """Two kernels in one call: the codes of a head do not depend on which one forms them, and its output only by
    the order of the sums."""
    n, H = 2, heads_for(queries, N, full=True)
    src = rand_qkv(1, n, N, 9000 + N)
    g, o = run(src, H, (1, 1, N))
    assert repeats_agree(g, n)
    pp = oracle.prep(*src, (1, 1, N))
    rows = np.arange(0, N, 5)
    assert_codes_equal(g[:n].cpu().numpy(), oracle.attention_codes(pp, rows), rows, f"{queries}")
    ref = oracle.attention(pp, rows)
    for h in (0, H // 2, H - 2, H - 1):   # the last heads are the other kernel's
        check_output(values(o[h:h + 1], 1)[:, rows], ref[h % n][None], f"{queries} head {h}")


@pytest.mark.parametrize("N", [300, 1000, 1500])
def test_a_head_alone_and_in_a_larger_call(N):
    """A head's codes are the same in every call; its output is reproducible for the same (B H, N), and between
    calls of different sizes differs by the order of its sums and of its block means' batches: before the
    rounding to bf16 by at most 2^-15 of the largest value (the means' two bf16 parts leave 2^-16 each), so by
    at most that and one bf16 step after it."""
    src = rand_qkv(1, 1, N, 9500 + N)
    alone = run(src, 1, (1, 1, N))
    assert all(torch.equal(a, b) for a, b in zip(alone, run(src, 1, (1, 1, N))))
    top = float(np.abs(S.bits_to_f32(src[2])).max())
    a = values(alone[1], 1)[0]
    for queries in (256, 128):
        g, o = run(src, heads_for(queries, N), (1, 1, N))
        assert torch.equal(g[0], alone[0][0])
        b = values(o, 1)[0]
        step = 2.0 ** (np.floor(np.log2(np.maximum(np.maximum(np.abs(a), np.abs(b)), 1e-30))) - 7)
        assert (np.abs(a - b) <= step + 2.0 ** -15 * top).all()
        assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(a)
