"""Evaluations whose y shares memory with u (the same array, or one shifted by a few rows) give
the bits of the evaluation into an array of its own, in every form."""
import numpy as np
import pytest

import paper_2311_03694_amd as rg
import romsynth

pytestmark = pytest.mark.gpu

DTS = ["fp64", "fp32", "bf16", "bf16x3"]


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _rom(form, N, R, dt, B):
    A = romsynth.stiffness_diag(N)
    rng = np.random.default_rng(N + R)
    if form == "pairs":
        lam, Af, Bf, Cf = romsynth.skew_cp_factors(N, R // 2, seed=N, cfg=90)
        return rg.Rom(N, 1e-3, 1e-3, A, lam=lam, Af=Af, Bf=Bf, Cf=Cf, dtype=dt, max_batch=B)
    if form == "general":
        Af, Bf, Cf = (rng.standard_normal((N, R)) for _ in range(3))
        return rg.Rom(N, 1e-3, 1e-3, A, lam=np.ones(R), Af=Af, Bf=Bf, Cf=Cf, dtype=dt, max_batch=B)
    if form == "svd":
        return rg.Rom(N, 1e-3, 1e-3, A, dtype=dt,
                      svd=(rng.standard_normal((N, R)), np.ones(R), rng.standard_normal((N, N, R))))
    return rg.Rom(N, 1e-3, 1e-3, A, C=rng.standard_normal((N, N, N)), dtype=dt, max_batch=B)


# one launch over one and several blocks of 16 rows (N = 16, 17, 37, 96), and the operators past it
@pytest.mark.parametrize("dt", DTS)
@pytest.mark.parametrize("form,N,R,B", [("general", 16, 8, 1), ("general", 17, 6, 1), ("general", 37, 40, 1),
                                        ("pairs", 37, 40, 1), ("pairs", 96, 24, 1), ("pairs", 64, 128, 1),
                                        ("dense", 40, 0, 1), ("svd", 40, 6, 1), ("general", 37, 40, 5),
                                        ("dense", 40, 0, 5)])
def test_y_shares_memory_with_u(torch_gpu, dt, form, N, R, B):
    torch = torch_gpu
    rom = _rom(form, N, R, dt, B)
    u = torch.tensor(romsynth.initial_u(N, range(B), cfg=91), dtype=torch.float64, device="cuda").reshape(-1)
    for call in (rg.rom_nonlinear, rg.rom_nonlinear_noalloc):
        for shift in (0, 1, -1, 16, -16, u.numel() - 1, u.numel()):
            print(f"[case] in place {form} N={N} R={R} B={B} {dt} shift={shift} {call.__name__}", flush=True)
            y = torch.empty_like(u)
            torch.cuda.synchronize()
            call(rom.handle, B, u, y)
            room = torch.zeros(3 * u.numel() + 32, dtype=torch.float64, device="cuda")
            at = u.numel() + 16
            room[at:at + u.numel()] = u
            torch.cuda.synchronize()
            call(rom.handle, B, room[at:at + u.numel()], room[at + shift:at + shift + u.numel()])
            torch.cuda.synchronize()
            assert torch.equal(room[at + shift:at + shift + u.numel()], y)
    rom.close()
