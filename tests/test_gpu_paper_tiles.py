"""Paper-form LLSA at the edges of its tile kernels: 16 channels of diagonal
keys (one tile of keys, two of queries) against one fewer and one more, and
windows at the edges of the band pass's staged rows (112 and 144 at d = 64;
112, 144 and 288 at d = 32)."""

import pytest

from test_gpu_llsa_paper import check, run, run_check_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,H,d,Lb,La,lengths", [
    (2, 150, 2, 64, 48, 16, (70, 150)),
    (2, 150, 2, 64, 79, 16, (1, 150)),   # the widest look-back of the one-pass forward
    (2, 150, 2, 64, 80, 16, (70, 150)),  # and one past it
    (2, 150, 3, 32, 64, 16, (16, 150)),
    (1, 17, 1, 64, 0, 16, "full"),
    (3, 9, 2, 32, 5, 16, (0, 9, 4)),     # look-ahead longer than the sequences
    (2, 90, 2, 64, 20, 15, (17, 90)),
    (2, 90, 2, 64, 20, 17, (17, 90)),
])
def test_forward_and_backward_around_16(oracle_mod, B, T, H, d, Lb, La, lengths):
    check(*run(oracle_mod, B, T, H, d, Lb, La, "bf16", 61, lengths, "unit"), "bf16")
    run_check_bwd(oracle_mod, B, T, H, d, Lb, La, 62, lengths, "unit", dtype="bf16")


@pytest.mark.parametrize("d,Lb,La", [
    (64, 40, 8),   # 112 rows
    (64, 41, 8),   # 144 rows (one sub-block more)
    (64, 32, 16), (64, 33, 16),
    (32, 40, 8), (32, 41, 8),
    (32, 48, 16), (32, 49, 16),   # 144, and past it
    (32, 192, 16),                # 288
])
def test_backward_staged_rows(oracle_mod, d, Lb, La):
    run_check_bwd(oracle_mod, 2, 210, 2, d, Lb, La, 63, (65, 210), "unit", dtype="bf16")
