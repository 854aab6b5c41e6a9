"""fscc_zgemm_noalloc plans on the host before it looks for a device: without a GPU a size that fits the static scratch
gets as far as that (FSCC_EHIP), one that does not is refused (FSCC_EINVAL).  No operand is touched."""
import ctypes

import pytest

import paper_2004_03682_amd as F

EINVAL, EHIP = -1, -4


@pytest.mark.parametrize("M,N,K,tB,status", [
    (1000, 10, 10, 0, EHIP), (0, 5, 5, 0, EHIP),
    # few columns of up to 2e8 rows: 16-byte tables of 256-row tiles, or of 128 x 16 ones
    (150_000_000, 3, 10, 0, EHIP), (200_000_000, 16, 32, 0, EHIP), (150_000_000, 16, 300, 0, EHIP),
    (16, 150_000_000, 300, 0, EHIP), (40_000, 40_000, 10, 0, EHIP),
    (200_000, 200_000, 10, 0, EINVAL)])
@pytest.mark.parametrize("split", [0, 1])
def test_default_form_fits_the_scratch_where_any_form_does(M, N, K, tB, status, split):
    torch = pytest.importorskip("torch")
    if torch.cuda.device_count() > 0:
        pytest.skip("without a GPU only: the operands do not exist")
    p = ctypes.c_void_p(64)
    r = F.lib().fscc_zgemm_noalloc(-1, 16, 0, tB, 0, 0, M, N, K, p, max(K, 1), p, max(K if tB else N, 1), p, max(N, 1),
                                   ctypes.c_double(1.0), ctypes.c_double(0.0), 0, split, None)
    assert r == status, F.lib().fscc_last_error(None).decode()
