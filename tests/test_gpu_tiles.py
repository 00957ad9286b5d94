"""The batched CP products over tiled operands: sizes around whole tiles, whole steps of each
format and whole rounds of the prefetch ring, evaluations and steps against the oracle."""
import numpy as np
import pytest

import oracle as orc
import paper_2311_03694_amd as rg
import romsynth
from helpers import TRAJ_TOL, check_eval, eval_bound_cp, rel

pytestmark = pytest.mark.gpu

# (N, R, B): one row and column; K of one step and less; rows and K past a tile or step by one;
# rings with one step, a full ring, one more; ranks whose padding to 8 is not one to 16
CASES = [(1, 1, 2), (7, 3, 17), (16, 16, 16), (17, 33, 33), (33, 40, 5), (128, 24, 16), (130, 257, 18), (520, 100, 3)]


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("N,R,B", CASES)
def test_cp_tiles(torch_gpu, dt, N, R, B):
    torch = torch_gpu
    print(f"[case] cp tiles N={N} R={R} B={B} {dt}", flush=True)
    rng = np.random.default_rng(N * 1000 + R)
    lam = 1.0 / np.arange(1, R + 1)
    Af, Bf, Cf = (rng.standard_normal((N, R)) / np.sqrt(N) for _ in range(3))
    U = romsynth.initial_u(N, range(B), cfg=62)
    ops = [lam, Af, Bf, Cf]
    Ur = U
    if dt == "bf16":                        # its products of rounded operands are exact
        lr, Ar, Br, Cr, Ur = (orc.round_bf16(a).reshape(np.shape(a)) for a in (lam, Af, Bf, Cf, U))
    else:
        lr, Ar, Br, Cr = ops
    for A in (romsynth.stiffness_diag(N), romsynth.stiffness_spd(N, 1, 62)):
        rom = rg.Rom(N, 1e-3, 1e-3, A, lam=lam, Af=Af, Bf=Bf, Cf=Cf, dtype=dt, max_batch=B)
        ud = torch.tensor(U, device="cuda")
        yd = torch.empty_like(ud)
        torch.cuda.synchronize()
        rg.rom_nonlinear(rom.handle, B, ud, yd)
        torch.cuda.synchronize()
        Y = yd.cpu().numpy()
        for b in range(B):
            check_eval(dt, Y[b], orc.nonlinear_cp(lr, Ar, Br, Cr, Ur[b]), eval_bound_cp(dt, lam, Af, Bf, Cf, U[b]))
        st = rom.state(U)
        st.step(6)
        u = st.u()
        for b in (0, B - 1):
            r = orc.run(N, 1e-3, 1e-3, A, 6, u0=U[b], lam=lam, Af=Af, Bf=Bf, Cf=Cf)
            assert rel(u[b], r["u_hist"][0]) < TRAJ_TOL[dt]
        st.close()
        rom.close()
