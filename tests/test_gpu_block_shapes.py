"""The reverse block kernel at the detected-mode and block-coordinate counts where
it changes form: 16 positions (the pivot's row and column on the vector unit), more
(two tiles), and two or three undetected modes (eight wavefronts up to four
detected modes, four beyond), with ragged chunks.  Checks, inputs and tolerances of
test_gpu_kernel_edges (at most 20 levels of sums over 23 terms here)."""
import pytest

import test_gpu_kernel_edges as E

pytestmark = pytest.mark.gpu

# cutoffs and how many of the first modes are undetected
SHAPES = [([9, 3, 2, 3, 2, 2, 2, 3], 1), ([4, 3, 2, 3, 2, 2, 2, 3], 2), ([3, 2, 3, 3, 2, 2, 3, 2], 3),   # 16 positions
          ([21, 2, 3, 2, 2, 2, 2, 2], 1), ([5] + [2] * 8, 1), ([3, 4] + [2] * 7, 2), ([3, 4] + [2] * 8, 2),
          ([3, 2, 3] + [2] * 6, 3), ([3, 2, 2] + [2] * 8, 3),                                            # more
          ([3, 5, 6], 2), ([7, 6, 3, 4], 2), ([2, 3, 2, 5], 3), ([4, 3, 3, 3, 2, 3], 2), ([3, 2, 2, 2, 3, 2, 3], 3),
          ([5, 4, 2, 3, 2, 3, 2], 2)]


@pytest.mark.parametrize("b_zero", [True, False])
@pytest.mark.parametrize("cut,undetected", SHAPES)
def test_reverse_block_forms(cut, undetected, b_zero):
    E.test_sweeps_agree(cut, ((1 << len(cut)) - 1) & ~((1 << undetected) - 1), b_zero)
