"""The attention kernels that a call's rows are dealt to (256, 128 or 32 queries per workgroup), at shapes
that take each of them alone and after full rounds of the 256-query one: attention of the heads on both
sides of every change against the CPU oracle, probability codes of the split-key kernel bit for bit, and
the output of a ragged last group."""
import numpy as np
import pytest

import oracle
import synthetic as S
from test_gpu_codes import assert_codes_equal, gpu_codes
from test_gpu_mx import rand_qkv
from test_gpu_parity import check_output, dev16

torch = pytest.importorskip("torch")
vc = pytest.importorskip("paper_2609_15810_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vc.lib()


@pytest.mark.parametrize("H,N,fmt,p_mode,heads", [
    (60, 300, "int8", 0, (0, 31, 59)),       # 128-query workgroups alone (180)
    (45, 1500, "int8", 0, (0, 42, 44)),      # 256 of 256 queries, then 109 groups of 32 from within head 42
    (55, 1500, "mxfp4", 1, (0, 42, 54)),     # 256 of 256 queries, then 148 of 128 from within head 42
    (128, 512, "int8", 1, (0, 127)),         # exactly one round of 256-query workgroups
    (3, 1025, "mxfp4", 0, (0, 1, 2)),        # 32-query groups alone, the last with one query, key tiles 1 or 2 per wave
])
def test_rows_dealt_to_each_kernel(H, N, fmt, p_mode, heads):
    Q, K, V = rand_qkv(1, H, N, 11 * H + N)
    qk = {"int8": vc.QK_INT8, "mxfp4": vc.QK_MXFP4}[fmt]
    A = vc.Attention(1, H, (1, 1, N), vc.make_opts(qk_fmt=qk, p_mode=p_mode), vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.prep(dev16(Q), dev16(K), dev16(V), perm=None)
    O = torch.full((1, H, N, 128), 0x7fc0, dtype=torch.int16, device="cuda")   # NaN: a row left out shows
    A.forward(O)
    torch.cuda.synchronize()
    o = S.bits_to_f32(O.cpu().numpy().view(np.uint16)).reshape(H, N, 128).astype(np.float64)
    assert np.isfinite(o).all()
    sel = list(heads)
    pp = oracle.prep(Q[:, sel], K[:, sel], V[:, sel], (1, 1, N), qk_fmt={"int8": oracle.QK_INT8, "mxfp4": oracle.QK_MXFP4}[fmt])
    rows = np.unique(np.concatenate([np.arange(0, N, 7), [N - 1]])).astype(np.int32)
    check_output(o[sel][:, rows], oracle.attention(pp, rows, p_mode=p_mode), f"{H}x{N} {fmt}")


@pytest.mark.parametrize("N", [64, 257, 1025, 2000])   # 64: not split; else one to two tiles per wave, waves without a tile
def test_split_key_codes(N):
    Q, K, V = rand_qkv(1, 2, N, 5 * N)
    g, O1, O2 = gpu_codes(Q, K, V, (1, 1, N))
    rows = np.arange(N)
    pp = oracle.prep(Q, K, V, (1, 1, N))
    assert_codes_equal(g, oracle.attention_codes(pp, rows), rows, f"N={N}")
    assert np.array_equal(O1, O2)


@pytest.mark.parametrize("low", [0, 1])
def test_split_key_domain_needs_all_keys_of_the_first_tile(low):
    """Rows whose first key tile has all scores of one lane half's keys below -2^27 (log2 units) and those of
    the other half at 0: their maximum is in the domain, so they are the method's result and not NaN."""
    N, H = 300, 2
    rng = np.random.default_rng(21 + low)
    half = (np.arange(N) >> 2) & 1                       # the lane half that holds a key's score
    k = np.where((half == low) & (np.arange(N) < 128), -1000.0, 0.0)
    Q = S.bf16_bits(np.full((1, H, N, 128), 1000.0, np.float32))
    K = S.bf16_bits(np.broadcast_to(k[None, None, :, None], (1, H, N, 128)).astype(np.float32))
    V = S.bf16_bits(rng.standard_normal((1, H, N, 128)).astype(np.float32))
    opt = dict(rope=False, hadamard=False, smooth_k=False)
    g, O1, O2 = gpu_codes(Q, K, V, (1, 1, N), sm_scale=1.0, **opt)
    pp = oracle.prep(Q, K, V, (1, 1, N), **opt)
    rows = np.arange(N)
    score = float(pp["q_scale"].flat[0] * pp["k_scale"].flat[0]) * -(127.0 ** 2) * 128 * np.log2(np.e)
    assert score < -(2.0 ** 27)                          # the premise: that half is beyond the domain's limit
    assert_codes_equal(g, oracle.attention_codes(pp, rows, sm_scale=1.0), rows, f"half {low}")
    o = S.bits_to_f32(O2.view(np.uint16)).reshape(H, N, 128).astype(np.float64)
    assert np.isfinite(o).all()
    check_output(o, oracle.attention(pp, rows, sm_scale=1.0), f"half {low}")
    assert np.array_equal(O1, O2)
