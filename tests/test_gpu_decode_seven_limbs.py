"""Decoding of seven-limb ciphertexts, the last count that takes a variant of its
own, at the ring sizes that test_gpu_decode.py leaves out.  Needs an MI355X."""
import pytest

import test_gpu_decode as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN", [13, 15])
def test_seven_limbs(logN):
    D.test_every_limb_count(logN, 7)
