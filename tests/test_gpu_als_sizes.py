"""CP-ALS and ALS-skew around the edges of the product's column groups and the inverse's
panels: every number of column tiles a block can hold, ranks that fill the last tile and
group or do not, tensors read in place and unfolded (ragged N, an address that is not a
multiple of 16 bytes), inverses of one to five panels, and the product past the kernel's
range (rows of more than 1000 columns)."""
import concurrent.futures as cf

import numpy as np
import pytest

import oracle as orc
import paper_2311_03694_amd as rg

pytestmark = pytest.mark.gpu
TOL = 1e-8          # a few sweeps of well-conditioned FP64 least squares: far above their rounding


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _device(torch, X, shift):
    """X on the device, `shift` doubles past the start of an allocation."""
    buf = torch.empty(X.size + shift, dtype=torch.float64, device="cuda")
    buf[shift:].copy_(torch.from_numpy(X.ravel()))
    return buf[shift:].view(X.shape)


def _rank(rng, N, R):
    """A noisy tensor of rank R and a first guess near its factors."""
    T = [rng.standard_normal((N, R)) for _ in range(3)]
    X = np.tensordot(T[0], T[1][:, None, :] * T[2][None, :, :], axes=(1, 2))
    X = X + 1e-3 * rng.standard_normal((N, N, N))
    return X, [t + 0.1 * rng.standard_normal(t.shape) for t in T]


# (N, R, shift): column tiles per block (of at most 6, fewer where the panel's rows are long)
# 1, 2, 3, 4, 5, 6, and more than one group of columns; N of whole 8-k steps (read in place
# unless shifted) and ragged; R of one to five 32-column panels, full and ragged
@pytest.mark.parametrize("N,R,shift", [(1, 1, 0), (8, 16, 0), (16, 17, 1), (24, 33, 0), (31, 64, 0), (40, 65, 1),
                                       (48, 96, 0), (56, 97, 0), (200, 72, 0), (203, 30, 0), (340, 40, 0)])
def test_als_sizes(torch_gpu, N, R, shift):
    print(f"[case] cp-als N={N} R={R} shift={shift}", flush=True)
    X, F0 = _rank(np.random.default_rng(N + R), N, R)
    Xd = _device(torch_gpu, X, shift)
    Fd = [torch_gpu.tensor(f, device="cuda") for f in F0]
    torch_gpu.cuda.synchronize()
    rg.rom_cp_als(N, R, Xd, *Fd, 2)
    torch_gpu.cuda.synchronize()
    F, _ = orc.als.cp_als(X, *F0, 2)
    for a, b in zip(Fd, F):
        assert np.max(np.abs(a.cpu().numpy() - b)) <= TOL * np.max(np.abs(b))


@pytest.mark.parametrize("N,P,shift", [(16, 8, 0), (24, 33, 1), (29, 48, 0), (80, 49, 0)])
def test_als_skew_sizes(torch_gpu, N, P, shift):
    print(f"[case] als-skew N={N} P={P} shift={shift}", flush=True)
    rng = np.random.default_rng(N + P)
    init = [rng.standard_normal((N, P)) for _ in range(3)]
    G = rng.standard_normal((N, N, N))
    X = G - G.transpose(2, 1, 0)
    Xd = _device(torch_gpu, X, shift)
    Fd = [torch_gpu.tensor(f, device="cuda") for f in init]
    torch_gpu.cuda.synchronize()
    rg.rom_cp_als_skew(N, P, Xd, *Fd, 2, 2, 0.5)
    torch_gpu.cuda.synchronize()
    F, _ = orc.als.als_skew(X, *init, sweeps=2, subiters=2, momentum=0.5)
    for a, b in zip(Fd, F):
        assert np.max(np.abs(a.cpu().numpy() - b)) <= TOL * np.max(np.abs(b))


def test_als_past_the_kernel(torch_gpu):
    """N = 1003: a column tile's panel no longer fits in LDS (the skinny product), one sweep
    against the same least squares in FP64 torch on the device."""
    torch = torch_gpu
    N, R = 1003, 3
    print(f"[case] cp-als N={N} R={R}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    F = [torch.randn(N, R, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    first = [f + 0.1 * torch.randn(N, R, dtype=torch.float64, device="cuda", generator=g) for f in F]
    X = torch.mm(F[0], (F[1][:, None, :] * F[2][None, :, :]).reshape(N * N, R).T.contiguous()).view(N, N, N)
    G = [f.clone() for f in first]
    torch.cuda.synchronize()
    rg.rom_cp_als(N, R, X, *G, 1)
    torch.cuda.synchronize()
    A = [f.clone() for f in first]
    gram = lambda a, b: (a.T @ a) * (b.T @ b)
    t = torch.mm(X.view(N * N, N), A[2]).view(N, N, R)
    A[0] = torch.linalg.solve(gram(A[1], A[2]), (t * A[1][None]).sum(1).T).T.contiguous()
    A[1] = torch.linalg.solve(gram(A[0], A[2]), (t * A[0][:, None]).sum(0).T).T.contiguous()
    t = torch.mm(X.view(N, N * N).T, A[0]).view(N, N, R)                 # rows (j, k)
    A[2] = torch.linalg.solve(gram(A[0], A[1]), (t * A[1][:, None]).sum(0).T).T.contiguous()
    for a, b in zip(G, A):
        assert float((a - b).abs().max()) <= TOL * float(b.abs().max())



def test_als_from_several_threads(torch_gpu):
    """Eight calls at once, more than there are stream pairs: those beyond run on the caller's
    stream alone, with the same results to the bit."""
    torch = torch_gpu
    rng = np.random.default_rng(9)
    N, R = 48, 70
    X, F0 = _rank(rng, N, R)
    Xd = _device(torch, X, 0)

    def fit(stream):
        G = [torch.tensor(f, device="cuda") for f in F0]
        torch.cuda.synchronize()
        rg.rom_cp_als(N, R, Xd, *G, 4, stream=stream)
        return G

    ref = fit(None)
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        out = list(ex.map(fit, [torch.cuda.Stream() for _ in range(8)]))
    torch.cuda.synchronize()
    for G in out:
        assert all(torch.equal(a, b) for a, b in zip(G, ref))
