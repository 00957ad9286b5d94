"""The folded dense tensor (one word per unordered pair j, k): every chunk shape, remainder
and column tile against the oracle, and the unfolded staging of tensors whose sums overflow."""
import numpy as np
import pytest

import oracle as orc
import paper_2311_03694_amd as rg
import romsynth
from helpers import check_eval, eval_bound_dense

pytestmark = pytest.mark.gpu

# one row and chunk, tile and chunk edges (16 rows, half and whole chunks of 32 and 64), odd
# and even numbers of chunks
SIZES = [1, 2, 15, 17, 31, 32, 33, 48, 49, 64, 65, 97, 128, 161, 200]


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _eval(torch, rom, U, call=None):
    ud = torch.tensor(U, dtype=torch.float64, device="cuda")
    yd = torch.empty_like(ud)
    torch.cuda.synchronize()
    (call or rg.rom_nonlinear)(rom.handle, ud.shape[0], ud, yd)
    torch.cuda.synchronize()
    return yd.cpu().numpy()


@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("N", SIZES)
def test_folded_evaluations(torch_gpu, dt, N):
    """One trajectory and batches (one and several column tiles, ragged) at every chunk edge;
    the tensor has no symmetry of its own."""
    print(f"[case] folded N={N} {dt}", flush=True)
    rng = np.random.default_rng(700 + N)
    C = rng.standard_normal((N, N, N)) / N
    U = romsynth.initial_u(N, range(70), cfg=61)
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype=dt, max_batch=70)
    ref = [orc.nonlinear_dense(C, u) for u in U]
    bound = [eval_bound_dense(dt, C, u) for u in U]
    for B, variants in ((1, (-1,)), (3, (-1,)), (33, (0, 1, 2)), (70, (-1, 9, 13))):
        for v in variants:
            rg.rom_set_tile(rom.handle, 1, v)
            Y = _eval(torch_gpu, rom, U[:B])
            for b in range(B):
                check_eval(dt, Y[b], ref[b], bound[b])


@pytest.mark.parametrize("dt", ["fp32", "bf16x3"])
@pytest.mark.parametrize("B", [1, 5])
def test_unfolded_where_sums_overflow(torch_gpu, dt, B):
    """Entries whose pair sums pass the format's largest value are staged unfolded: the
    evaluation of small u stays finite and equals the oracle's."""
    N = 70
    rng = np.random.default_rng(5)
    C = rng.standard_normal((N, N, N))
    C[3, 10, 40] = C[3, 40, 10] = 2.5e38
    U = 1e-19 * rng.standard_normal((B, N))
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype=dt, max_batch=B)
    Y = _eval(torch_gpu, rom, U)
    assert np.all(np.isfinite(Y))
    for b in range(B):
        check_eval(dt, Y[b][3:4], orc.nonlinear_dense(C, U[b])[3:4], eval_bound_dense(dt, C, U[b]))


def test_bounded_workspace_takes_fewer_partial_tiles(torch_gpu):
    """rom_nonlinear_noalloc accepts a batch whose usual partial tiles exceed its scratch."""
    N, B = 128, 8192
    rng = np.random.default_rng(6)
    C = rng.standard_normal((N, N, N)) / N
    U = romsynth.initial_u(N, range(B), cfg=61)
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype="fp64", max_batch=B)
    Y = _eval(torch_gpu, rom, U)
    Z = _eval(torch_gpu, rom, U, rg.rom_nonlinear_noalloc)
    for b in (0, 17, 4097, B - 1):
        ref, bound = orc.nonlinear_dense(C, U[b]), eval_bound_dense("fp64", C, U[b])
        check_eval("fp64", Y[b], ref, bound)
        check_eval("fp64", Z[b], ref, bound)
