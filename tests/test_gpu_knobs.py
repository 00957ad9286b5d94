"""rom_set_tile reaches every variant of the contractions and of the CP products, and the sums it
changes stay within the format's bound."""
import numpy as np
import pytest

import oracle as orc
import paper_2311_03694_amd as rg
import romsynth
from helpers import check_eval, eval_bound_dense

pytestmark = pytest.mark.gpu

FOLD_VARIANTS = 21                                      # three shapes, the planned split and six fixed ones


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _eval(torch, rom, U):
    ud = torch.tensor(U, dtype=torch.float64, device="cuda")
    yd = torch.empty_like(ud)
    torch.cuda.synchronize()
    rg.rom_nonlinear(rom.handle, ud.shape[0], ud, yd)
    torch.cuda.synchronize()
    return yd.cpu().numpy()


@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("kind,B", [(0, 1), (1, 20)])
def test_dense_knobs(torch_gpu, dt, kind, B):
    print(f"[case] dense knob {kind} {dt}", flush=True)
    N = 90
    assert rg.rom_tile_count(1) >= FOLD_VARIANTS
    C = np.random.default_rng(kind).standard_normal((N, N, N)) / N
    U = romsynth.initial_u(N, range(B), cfg=95)
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype=dt, max_batch=B)
    Cr, Ur = (orc.round_bf16(a).reshape(np.shape(a)) for a in (C, U)) if dt == "bf16" else (C, U)
    first = _eval(torch_gpu, rom, U)
    for v in range(rg.rom_tile_count(kind)):
        rg.rom_set_tile(rom.handle, kind, v)
        Y = _eval(torch_gpu, rom, U)
        for b in range(0, B, 7):
            check_eval(dt, Y[b], orc.nonlinear_dense(Cr, Ur[b]), eval_bound_dense(dt, C, U[b]))
    rg.rom_set_tile(rom.handle, kind, -1)
    assert np.array_equal(first, _eval(torch_gpu, rom, U))


# value 0 takes two column tiles a block in the projections here
@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
def test_cp_tile_widths(torch_gpu, dt):
    """The four column-tile choices of the CP products (0 .. 3) give the same bits."""
    print(f"[case] cp tile widths {dt}", flush=True)
    N, R, B = 900, 1000, 64
    rng = np.random.default_rng(3)
    F = [rng.standard_normal((N, R)) for _ in range(3)]
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), lam=np.ones(R), Af=F[0], Bf=F[1], Cf=F[2], dtype=dt,
                 max_batch=B)
    U = romsynth.initial_u(N, range(B), cfg=96)
    Y = []
    for v in (-1, 0, 1, 2, 3):
        for kind in (2, 3):
            rg.rom_set_tile(rom.handle, kind, v)
        Y.append(_eval(torch_gpu, rom, U))
    assert np.all(np.isfinite(Y[0])) and all(np.array_equal(Y[0], y) for y in Y[1:])
