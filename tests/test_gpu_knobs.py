"""rom_set_tile reaches every variant of the CP products."""
import numpy as np
import pytest

import paper_2311_03694_amd as rg
import romsynth

pytestmark = pytest.mark.gpu

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
