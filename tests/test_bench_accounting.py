"""What bench.py counts as the momentum kernel's traffic: one image of U where the library keeps X^T alone, two where it keeps X as well."""
import pytest

from bench import momentum_bytes

EL = 12.0   # bf16 gradient, fp32 momentum in and out, one bf16 image


@pytest.mark.parametrize("shapes,want", [
    ([(256, 512)] * 6, 6 * 256 * 512 * EL),                        # 1536 rows in all
    ([(256, 512)] * 5, 5 * 256 * 512 * (EL + 2)),                  # fewer: X as well
    ([(300, 77), (77, 300)], 2 * 300 * 77 * (EL + 2)),             # one batch of 512 padded rows
    ([(25600, 5120)] * 4, 4 * 25600 * 5120 * EL),                  # merged steps
    ([(1024, 1024), (1024, 2048)], 3 * 1024 * 1024 * EL),          # two classes of one run: 2048 rows
    ([(1024, 1024), (5120, 13824)], 1024 * 1024 * (EL + 2) + 5120 * 13824 * EL),   # a run of its own each
], ids=["six", "five", "transposed", "merged", "one run", "two runs"])
def test_images_of_u(shapes, want):
    assert momentum_bytes(shapes, 1, 2, 5, True) == want


def test_both_images_without_the_x_t_product():
    assert momentum_bytes([(4096, 4096)], 1, 2, 0, True) == 4096 * 4096 * (EL + 2)
    assert momentum_bytes([(4096, 4096)], 1, 4, 5, False) == 4096 * 4096 * (4 + 8 + 8)
