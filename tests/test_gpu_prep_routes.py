"""The two statistics kernels of the preprocessing and the two ways of storing codes on both sides of the
line between them (1280 blocks of 128 rows over all heads): codes, scales and means of the first, a middle and the last head bit for bit
against the CPU oracle, ragged last blocks, with and without permutation, rotation and centering."""
import numpy as np
import pytest

import oracle
import synthetic as S
from layouts import untile_qk, untile_v
from test_gpu_mx import rand_qkv
from test_gpu_parity import assert_prep_equal, dev16, dev32

torch = pytest.importorskip("torch")
vc = pytest.importorskip("paper_2609_15810_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vc.lib()


@pytest.mark.parametrize("H", [640, 644])   # 1280 blocks; 1288, waves of four blocks with one or two of them past the end
@pytest.mark.parametrize("grid,perm,opt", [
    ((2, 9, 11), True, {}),                                     # N = 198: rows wrap within a batch, ragged block
    ((1, 1, 129), True, dict(smooth_v=False)),                  # a last block of one row
    ((16, 16, 1), False, dict(smooth_k=False)),                 # full blocks, one column per row
    ((2, 16, 8), False, dict(rope=False, hadamard=False)),
])
def test_both_sides_of_the_line(H, grid, perm, opt):
    N = grid[0] * grid[1] * grid[2]
    sel = [0, H // 2, H - 1]
    Qs, Ks, Vs = rand_qkv(1, 3, N, N + len(opt))
    ps = S.random_perm(N, N, 1, 3)
    full = lambda x: np.concatenate([x[:, :1], np.repeat(x[:, 1:2], H - 2, 1), x[:, 2:]], 1)   # heads 1 .. H - 2 alike
    A = vc.Attention(1, H, grid, vc.make_opts(**opt), vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.prep(dev16(full(Qs)), dev16(full(Ks)), dev16(full(Vs)), perm=dev32(full(ps)) if perm else None)
    torch.cuda.synchronize()
    P = A.prepped
    pick = lambda t: t[:, sel].contiguous().cpu().numpy()
    got = dict(q=untile_qk(pick(P.q)), q_scale=pick(P.q_scale), k=untile_qk(pick(P.k)), k_scale=pick(P.k_scale),
               k_mean=pick(P.k_mean), v=untile_v(pick(P.v)), v_scale=pick(P.v_scale), v_mean=pick(P.v_mean).view(np.uint16))
    assert_prep_equal(got, oracle.prep(Qs, Ks, Vs, grid, perm=ps if perm else None, **opt), f"H={H} {grid}")


@pytest.mark.parametrize("fmt", ["fp8", "mxfp4"])
def test_score_formats_past_the_line(fmt):
    from layouts import untile_f8, untile_mx_codes, untile_mx_scales
    H, N, grid = 800, 198, (2, 9, 11)
    sel = [0, 400, 799]
    Qs, Ks, Vs = rand_qkv(1, 3, N, 77)
    full = lambda x: np.concatenate([x[:, :1], np.repeat(x[:, 1:2], H - 2, 1), x[:, 2:]], 1)
    A = vc.Attention(1, H, grid, vc.make_opts(qk_fmt={"fp8": vc.QK_FP8, "mxfp4": vc.QK_MXFP4}[fmt]),
                     vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.prep(dev16(full(Qs)), dev16(full(Ks)), dev16(full(Vs)), perm=None)
    torch.cuda.synchronize()
    P = A.prepped
    u8 = lambda t: t[:, sel].contiguous().cpu().numpy().view(np.uint8)
    o = oracle.prep(Qs, Ks, Vs, grid, qk_fmt={"fp8": oracle.QK_FP8, "mxfp4": oracle.QK_MXFP4}[fmt])
    if fmt == "fp8":
        pairs = [(untile_f8(u8(P.q)), o["q"].view(np.uint8)), (untile_f8(u8(P.k)), o["k"].view(np.uint8))]
    else:
        pairs = [(untile_mx_codes(u8(P.q)), o["q_mx"]), (untile_mx_scales(u8(P.q_mx_scale)), o["q_mxs"]),
                 (untile_mx_codes(u8(P.k)), o["k_mx"]), (untile_mx_scales(u8(P.k_mx_scale)), o["k_mxs"])]
    pairs.append((untile_v(u8(P.v)), o["v"]))
    for i, (g, r) in enumerate(pairs):
        assert np.array_equal(g, r), (fmt, i)


@pytest.mark.parametrize("H", [2, 800])
def test_infinity_in_the_last_row_of_a_ragged_block(H):
    """The rows that pad a ragged block repeat its last row and stay out of its sums, whatever they hold."""
    N, grid = 198, (2, 9, 11)
    V = np.repeat(rand_qkv(1, 1, N, 5)[2], H, 1)
    V[0, :, N - 1, 3] = 0x7f80   # +inf
    Q, K = np.zeros_like(V), np.zeros_like(V)
    A = vc.Attention(1, H, grid, vc.make_opts(), vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.prep(dev16(Q), dev16(K), dev16(V), perm=None)
    torch.cuda.synchronize()
    m = A.prepped.v_mean.cpu().numpy().view(np.uint16)
    o = oracle.prep(Q[:, :1], K[:, :1], V[:, :1], grid)["v_mean"]
    assert o[0, 0, 1, 3] == 0x7f80
    assert all(np.array_equal(m[0, h], o[0, 0]) for h in range(H))


@pytest.mark.parametrize("N,opt", [(2048, {}), (2049, {}), (1921, dict(smooth_k=False)), (2177, dict(smooth_v=False)), (127, {})])
def test_head_statistics_folded_and_not(N, opt):
    """16 and 17 blocks per head: the quantization forms the key mean and value scales itself, or reads them."""
    Q, K, V = rand_qkv(1, 2, N, 3 * N)
    V[0, 1, :, 5] = V[0, 1, 0, 5]   # a constant channel: zero residual, scale 1
    perm = S.random_perm(N, N, 1, 2)
    A = vc.Attention(1, 2, (1, 1, N), vc.make_opts(**opt), vc.make_group_opts(mode=vc.GROUP_IDENTITY))
    A.ws.fill_(0x5a)
    A.prep(dev16(Q), dev16(K), dev16(V), perm=dev32(perm))
    torch.cuda.synchronize()
    P = A.prepped
    got = dict(q=untile_qk(P.q.cpu().numpy()), q_scale=P.q_scale.cpu().numpy(), k=untile_qk(P.k.cpu().numpy()),
               k_scale=P.k_scale.cpu().numpy(), k_mean=P.k_mean.cpu().numpy(), v=untile_v(P.v.cpu().numpy()),
               v_scale=P.v_scale.cpu().numpy(), v_mean=P.v_mean.cpu().numpy().view(np.uint16))
    assert_prep_equal(got, oracle.prep(Q, K, V, (1, 1, N), perm=perm, **opt), f"N={N}")
