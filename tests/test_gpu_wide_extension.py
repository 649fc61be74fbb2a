"""GPU: lines whose extension (blend points and the padding to a length of
factors 2, 3, 5) is longer than the 64 lanes of a wave, in the split line
kernel, against the FP64 oracle at the bars of the other line lengths."""
import pytest

from test_gpu_line_splits import test_split_kernel_matches_oracle as check

pytestmark = pytest.mark.gpu


# 1000 -> 1080 (80 extension points), 655 -> 720 (65), 788 -> 864 (76)
@pytest.mark.parametrize("nx,ny", [(1000, 12), (12, 655), (788, 13)])
def test_wide_extension_matches_oracle(nx, ny):
    check(nx, ny, 5, 25)
