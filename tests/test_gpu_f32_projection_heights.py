"""The fp32 projection on tiles of 64 rows, which launches of more than 768 tiles of 16 rows take (the
shapes of the general test run on 16) unless there would be more than 256 of them, and at the counts
between the two."""

import pytest

from tests.test_gpu_f32_tiles import test_projection as check_projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,hq,hkv,d,hid", [
    (384, 8, 4, 64, 136),     # 32 column tiles x 24: exactly 768
    (385, 8, 4, 64, 136),
    (512, 8, 4, 64, 136),     # exactly 1024, and 256 of 64 rows
    (513, 8, 4, 64, 136), (1025, 5, 5, 48, 40),
    (672, 4, 4, 64, 136),     # 24 x 42, and 264 of 64 rows
    (673, 4, 4, 64, 136)])    # 24 x 43
def test_heights(gpu_device, m, hq, hkv, d, hid):
    check_projection(gpu_device, m, hq, hkv, d, hid)
