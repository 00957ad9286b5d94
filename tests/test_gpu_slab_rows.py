"""SVD slabs past the size of the tiled storage: the stream over rows in every format, alone and in
a mixed launch, and the tiled storage where the slab weights fill the row stream's LDS."""
import numpy as np
import pytest

import oracle as orc
import paper_2311_03694_amd as rg
import romsynth
from helpers import EPS_OP, U_ACC, check_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# a little over 200 MB of slab words; N odd, a whole number of 16 rows, and the most weights that
# rom_create_svd accepts (u and they fill the row stream's 64 KB: tiled)
@pytest.mark.parametrize("dt,N,R", [("fp64", 129, 1507), ("fp32", 176, 1620), ("bf16", 201, 2479), ("bf16x3", 131, 2915),
                                    ("fp64", 64, 8128)])
def test_large_slabs(torch_gpu, dt, N, R):
    print(f"[case] slab rows N={N} R={R} {dt}", flush=True)
    assert N * N * R * {"fp64": 8, "fp32": 4, "bf16": 2, "bf16x3": 4}[dt] > 200e6
    torch = torch_gpu
    rng = np.random.default_rng(N + R)
    U, sig = rng.standard_normal((N, R)), 1.0 / np.arange(1, R + 1)
    V = rng.standard_normal((N, N, R), dtype=np.float32).astype(np.float64)
    u = romsynth.initial_u(N, [2], cfg=63)[0]
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), svd=(U, sig, V), dtype=dt)
    ud = torch.tensor(u, dtype=torch.float64, device="cuda")
    yd = torch.empty_like(ud)
    torch.cuda.synchronize()
    rg.rom_nonlinear(rom.handle, 1, ud, yd)
    torch.cuda.synchronize()
    Ur, sr, Vr, ur = U, sig, V, u
    if dt == "bf16":
        Ur, sr, Vr, ur = (orc.round_bf16(a).reshape(np.shape(a)) for a in (U, sig, V, u))
    # magnitudes sum_r sum_k |V_ikr| |u_k| sigma_r (|U|^T |u|)_r of the terms of y_i, their
    # operands' error (w is itself a product of three, and a sum of N terms) and the sum of N R
    mag = (np.abs(V).reshape(N * N, R) @ (sig * (np.abs(U).T @ np.abs(u)))).reshape(N, N) @ np.abs(u)
    bound = 2.0 * float(np.linalg.norm(mag)) * (EPS_OP[dt] + 4.0 * np.sqrt(N * R) * U_ACC[dt] + 4.0 * np.sqrt(N) * U_ACC[dt])
    check_eval(dt, yd.cpu().numpy(), orc.nonlinear_svd(Ur, sr, Vr, ur), bound)
    # alone, and in a mixed launch beside a small CP state: the same bits
    F = [rng.standard_normal((20, 4)) for _ in range(3)]
    cp = rg.Rom(20, 1e-3, 1e-3, romsynth.stiffness_diag(20), lam=np.ones(4), Af=F[0], Bf=F[1], Cf=F[2], dtype=dt)
    sa, sb, sc = rom.state(u[None]), rom.state(u[None]), cp.state(romsynth.initial_u(20, [1], cfg=63)[0][None])
    sa.step(7)
    rg.rom_step_multi([rom.handle, cp.handle], [sb.handle, sc.handle], 7)
    ga, gb = rg.rom_state_get(rom.handle, sa.handle), rg.rom_state_get(rom.handle, sb.handle)
    assert all(np.array_equal(x, y) for x, y in zip(ga[:2], gb[:2])) and np.all(np.isfinite(ga[0]))
