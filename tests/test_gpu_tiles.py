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


@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("N,R,skew", [(1, 1, False), (1, 2, True), (9, 5, False), (37, 40, True), (37, 39, False),
                                      (64, 80, True), (64, 82, True), (40, 41, False), (130, 14, True)])
def test_cp_small_evaluation(torch_gpu, dt, N, R, skew):
    """One trajectory around the largest operator that is evaluated in one launch, general and
    pair form (ranks whose padding the pair form writes itself)."""
    torch = torch_gpu
    print(f"[case] cp small N={N} R={R} {dt}", flush=True)
    rng = np.random.default_rng(N * 100 + R)
    if skew:
        lam, Af, Bf, Cf = romsynth.skew_cp_factors(N, R // 2, seed=R, cfg=62)
    else:
        lam = 1.0 / np.arange(1, R + 1)
        Af, Bf, Cf = (rng.standard_normal((N, R)) / np.sqrt(N) for _ in range(3))
    u = romsynth.initial_u(N, [3], cfg=62)[0]
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), lam=lam, Af=Af, Bf=Bf, Cf=Cf, dtype=dt)
    ud = torch.tensor(u, device="cuda")
    out = []
    for form in ((-1, 0) if skew else (-1,)):
        rg.rom_set_tile(rom.handle, 4, form)
        yd = torch.empty_like(ud)
        torch.cuda.synchronize()
        rg.rom_nonlinear(rom.handle, 1, ud, yd)
        torch.cuda.synchronize()
        out.append(yd.cpu().numpy())
    assert all(np.array_equal(out[0], y) for y in out)
    ops = [lam, Af, Bf, Cf, u]
    if dt == "bf16":
        ops = [orc.round_bf16(a).reshape(np.shape(a)) for a in ops]
    check_eval(dt, out[0], orc.nonlinear_cp(*ops), eval_bound_cp(dt, lam, Af, Bf, Cf, u))
