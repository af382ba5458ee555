"""Grouping kernels at their edges against the CPU oracle, bit for bit: the one-workgroup-per-head
route (N <= 1024) and the multi-workgroup one around their boundary, ragged 32-token steps, one or two
cluster blocks (k <= 32, k > 32), no update at all (iters = 0), warm starts, several steps per workgroup
(many heads), and heads whose values are all equal (every distance ties)."""
import numpy as np
import pytest

import oracle
import synthetic as S

torch = pytest.importorskip("torch")
vc = pytest.importorskip("paper_2609_15810_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vc.lib()


def values(H, N, seed):
    rng = np.random.default_rng(seed)
    centers = rng.standard_normal((H, 9, 128)) * 2.0
    x = centers[np.arange(H)[:, None], rng.integers(0, 9, (H, N))] + 0.6 * rng.standard_normal((H, N, 128))
    x[0] = x[0, :1]   # one head of equal tokens: all distances tie
    return S.bf16_bits(x.astype(np.float32))[None]


@pytest.mark.parametrize("H,N,k,iters,warm", [
    (2, 1, 1, 2, False), (2, 31, 31, 3, False), (3, 257, 32, 4, False), (2, 1024, 64, 3, True), (2, 1023, 33, 0, False),
    (2, 1025, 32, 0, True), (2, 1025, 32, 1, False), (3, 1281, 64, 3, False), (2, 2049, 7, 5, True), (2, 3000, 33, 4, False),
    (300, 1100, 8, 2, False),   # two workgroups' worth of steps per head
])
def test_group_edges(H, N, k, iters, warm):
    V = values(H, N, 7 * N + k)
    cent = np.random.default_rng(k).standard_normal((1, H, k, 128)).astype(np.float32) if warm else None
    A = vc.Attention(1, H, (1, 1, N), gopts=vc.make_group_opts(k=k, iters=iters, warm_start=warm))
    A.ws.fill_(0x5a)   # nothing of the workspace is assumed clear
    if warm:
        A.centroids.copy_(torch.from_numpy(cent))
    A.group(torch.from_numpy(V.view(np.int16)).cuda(), warm_start=warm)
    torch.cuda.synchronize()
    g = oracle.group(V, (1, 1, N), k=k, iters=iters, warm_start=warm, cent_in=cent)
    for name in ("labels", "perm", "inv_perm"):
        assert np.array_equal(getattr(A, name).cpu().numpy(), g[name]), name
    assert np.array_equal(A.centroids.cpu().numpy().view(np.uint32), np.asarray(g["centroids"], np.float32).view(np.uint32))


@pytest.mark.parametrize("H,N,k,iters", [(2, 700, 32, 3), (2, 1025, 64, 3), (1, 1026, 1, 2), (3, 2050, 33, 1), (5, 4097, 7, 4)])
def test_workspace_of_exactly_its_size(H, N, k, iters):
    """Nothing behind the workspace is written, and what its parts hold suffices."""
    V = values(H, N, 3 * N + k)
    A = vc.Attention(1, H, (1, 1, N), gopts=vc.make_group_opts(k=k, iters=iters))
    need = vc.workspace_size(A.shape, None, A.gopts)
    whole = torch.full((need + 65536,), 0x5a, dtype=torch.uint8, device="cuda")
    A.ws = whole[:need]
    A.group(torch.from_numpy(V.view(np.int16)).cuda())
    torch.cuda.synchronize()
    assert (whole[need:] == 0x5a).all()
    g = oracle.group(V, (1, 1, N), k=k, iters=iters)
    for name in ("labels", "perm", "inv_perm"):
        assert np.array_equal(getattr(A, name).cpu().numpy(), g[name]), name
    assert np.array_equal(A.centroids.cpu().numpy().view(np.uint32), np.asarray(g["centroids"], np.float32).view(np.uint32))
