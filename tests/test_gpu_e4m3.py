"""The BF16-refined form's low-plane conversion as the kernel does it."""
import ctypes

import pytest

from tests import hip

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_codes_of_every_float():
    """Every float of size up to 448 (and the byte each value of four goes to) against
    f32_to_e4m3, which the CPU test holds to the format's definition; zeros of either sign."""
    bad = torch.zeros(2, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert hip.load().e4m3_codes(ctypes.c_void_p(bad.data_ptr())) == 0
    n, pattern = bad.tolist()
    assert n == 0, (n, hex(pattern & 0xFFFFFFFF))
