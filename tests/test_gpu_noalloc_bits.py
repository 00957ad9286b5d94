"""rom_nonlinear_noalloc gives rom_nonlinear's bits also where the batch's own plan exceeds the
fixed scratch: folded contractions then run in parts, CP batches in slices, in place too."""
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


def _check(torch, rom, N, B):
    rng = np.random.default_rng(B)
    u = torch.tensor(rng.standard_normal((B, N)) / N, device="cuda")
    y, z = torch.full_like(u, float("nan")), torch.full_like(u, float("nan"))
    torch.cuda.synchronize()
    rg.rom_nonlinear(rom.handle, B, u, y)
    rg.rom_nonlinear_noalloc(rom.handle, B, u, z)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(y).all()) and torch.equal(y, z)
    for shift in (0, N, -N):                             # y over u, a trajectory on, one back
        room = torch.zeros((B + 2, N), dtype=torch.float64, device="cuda")
        room[1:B + 1] = u
        torch.cuda.synchronize()
        flat = room.reshape(-1)
        rg.rom_nonlinear_noalloc(rom.handle, B, flat[N:N + B * N], flat[N + shift:N + shift + B * N])
        torch.cuda.synchronize()
        assert torch.equal(flat[N + shift:N + shift + B * N].reshape(B, N), y)
    rom.close()


# the largest batches served (whole tiles and a ragged rest) of tensors cut into few and many parts
@pytest.mark.parametrize("dt,N,B", [("fp64", 128, 8192), ("fp64", 33, 20011), ("fp32", 128, 10000), ("fp32", 321, 3001),
                                    ("bf16x3", 200, 6000), ("bf16", 128, 9000)])
def test_dense_in_parts(torch_gpu, dt, N, B):
    print(f"[case] noalloc bits dense N={N} B={B} {dt}", flush=True)
    C = np.random.default_rng(N).standard_normal((N, N, N)) / N
    _check(torch_gpu, rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype=dt, max_batch=B), N, B)


# knobs: CP products of k_gemm (-1) and on the LDS tiles (4); sizes whose tiled copies outgrow the rows
@pytest.mark.parametrize("dt,N,R,B,knob", [("bf16x3", 5, 8, 180000, -1), ("bf16x3", 5, 8, 180001, 4),
                                           ("fp32", 40, 48, 30000, -1), ("fp64", 40, 48, 15000, 4)])
def test_cp_in_slices(torch_gpu, dt, N, R, B, knob):
    print(f"[case] noalloc bits cp N={N} R={R} B={B} {dt} knob={knob}", flush=True)
    rng = np.random.default_rng(N)
    F = [rng.standard_normal((N, R)) for _ in range(3)]
    rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), lam=np.ones(R), Af=F[0], Bf=F[1], Cf=F[2], dtype=dt,
                 max_batch=B)
    for kind in (2, 3):
        rg.rom_set_tile(rom.handle, kind, knob)
    _check(torch_gpu, rom, N, B)


@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
def test_every_dense_variant(torch_gpu, dt):
    """Each tile choice of the batched contraction, the index past the BF16 kernels' own included."""
    N, B = 70, 20
    C = np.random.default_rng(N).standard_normal((N, N, N)) / N
    for v in range(rg.rom_tile_count(1)):
        print(f"[case] noalloc bits dense N={N} B={B} {dt} variant {v}", flush=True)
        rom = rg.Rom(N, 1e-3, 1e-3, romsynth.stiffness_diag(N), C=C, dtype=dt, max_batch=B)
        rg.rom_set_tile(rom.handle, 1, v)
        _check(torch_gpu, rom, N, B)
