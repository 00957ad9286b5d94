"""The server admits operators by an estimate of their device bytes: it covers what rom_create and
the start-up state hold, in every kind and format, and little more."""
import pytest

from paper_2311_03694_amd.serve import RomBackend

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# N = 300 and 380: BF16 tensors on both sides of 100 MB; 65 and 130: ragged tiles and chunks
@pytest.mark.parametrize("kind", ["dense", "cp"])
@pytest.mark.parametrize("dt", ["fp64", "fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("N", [65, 130, 300, 380])
def test_operator_estimate_covers_the_context(torch_gpu, kind, dt, N):
    print(f"[case] operator bytes {kind} N={N} {dt}", flush=True)
    be = RomBackend(pool_slots=16)
    key = (N, 1, kind, dt)
    op, held = be.create_op(key)
    est = be.estimate_op_bytes(key)
    be.destroy_op(op)
    # the operators are counted exactly; the workspace, the slack of the allocations and the state
    # are covered by 1 MB and the state's term
    assert held <= est <= held + (2 << 20), (held, est)
