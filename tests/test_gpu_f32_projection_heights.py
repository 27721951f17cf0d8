"""The fp32 projection on tiles of 64 rows, which launches of more than 1024 tiles of 16 rows take (the
shapes of the general test run on 16), and at the count between the two."""

import pytest

from tests.test_gpu_f32_tiles import test_projection as check_projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,hq,hkv,d,hid", [
    (512, 8, 4, 64, 136),     # 32 column tiles x 32: exactly 1024
    (513, 8, 4, 64, 136), (1025, 5, 5, 48, 40)])
def test_heights(gpu_device, m, hq, hkv, d, hid):
    check_projection(gpu_device, m, hq, hkv, d, hid)
