"""CP-ALS on both sides of the product kernel's range: the panel of one 16-column tile takes 1 KB of
LDS per 8 columns of the unfolding, all 160 KB of it at N = 1280; longer rows go through the
skinny product, with a transposed factor and padded unfoldings."""
import pytest

import paper_2311_03694_amd as rg

pytestmark = pytest.mark.gpu
TOL = 1e-8          # one sweep of well-conditioned FP64 least squares: far above its rounding


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# the largest panel (whole rows; ragged: unfolded first), and the skinny product with a ragged
# last row tile (N^2 = 1281^2 is not a multiple of 16) and with whole ones; one and two column tiles
@pytest.mark.parametrize("N,R", [(1280, 18), (1275, 3), (1281, 3), (1288, 18)])
def test_als_at_the_panel_limit(torch_gpu, N, R):
    torch = torch_gpu
    print(f"[case] cp-als N={N} R={R}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    F = [torch.randn(N, R, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    first = [f + 0.1 * torch.randn(N, R, dtype=torch.float64, device="cuda", generator=g) for f in F]
    X = torch.mm(F[0], (F[1][:, None, :] * F[2][None, :, :]).reshape(N * N, R).T.contiguous()).view(N, N, N)
    G = [f.clone() for f in first]
    torch.cuda.synchronize()
    rg.rom_cp_als(N, R, X, *G, 1)
    torch.cuda.synchronize()
    A = [f.clone() for f in first]
    gram = lambda a, b: (a.T @ a) * (b.T @ b)
    t = torch.mm(X.view(N * N, N), A[2]).view(N, N, R)                   # rows (i, j)
    A[0] = torch.linalg.solve(gram(A[1], A[2]), (t * A[1][None]).sum(1).T).T.contiguous()
    A[1] = torch.linalg.solve(gram(A[0], A[2]), (t * A[0][:, None]).sum(0).T).T.contiguous()
    t = torch.mm(X.view(N, N * N).T, A[0]).view(N, N, R)                 # rows (j, k)
    A[2] = torch.linalg.solve(gram(A[0], A[1]), (t * A[1][:, None]).sum(0).T).T.contiguous()
    for a, b in zip(G, A):
        assert float((a - b).abs().max()) <= TOL * float(b.abs().max())
    del X, t
    torch.cuda.empty_cache()
