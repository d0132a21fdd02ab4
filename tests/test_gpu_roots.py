"""The projections' shortened reciprocal and square root against IEEE
rounding: the binary32 specification of the binning divides and takes roots,
and every bit of a key, a rectangle or a radius depends on them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RCP, SQRT = 0, 1


def bits(x):
    return int(np.float32(x).view(np.uint32))


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_25459_amd import gsr
    r = gsr.Renderer(0)
    yield r
    r.close()


def _check(R, root, first, count):
    x = (np.arange(count, dtype=np.uint32) + np.uint32(first)).view(np.float32)
    ref = np.sqrt(x) if root == SQRT else np.float32(1.0) / x
    bad = np.nonzero(R.debug_roots(root, first, count).view(np.uint32) != ref.view(np.uint32))[0]
    assert bad.size == 0, f"{bad.size} of {count} from 0x{first:08x}: first x = {float(x[bad[0]]).hex()}"


@pytest.mark.parametrize("e", [-126, -125, -1, 0, 1, 125])
def test_reciprocal_of_every_mantissa(R, e):
    """All 2^23 mantissas (and the next power of two), at both ends of the range too."""
    _check(R, RCP, bits(2.0 ** e), (1 << 23) + 1)


@pytest.mark.parametrize("e", [-100, -99, -1, 0, 1, 126, 127])
def test_square_root_of_every_mantissa(R, e):
    """All 2^23 mantissas for either parity of the exponent, at both ends of the range too."""
    _check(R, SQRT, bits(2.0 ** e), 1 << 23)


@pytest.mark.parametrize("root,lo,hi", [(RCP, -126, 125), (SQRT, -100, 127)])
def test_roots_at_every_exponent(R, root, lo, hi):
    """The smallest and the largest mantissas of every binade of the range."""
    for e in range(lo, hi + 1):
        first = bits(2.0 ** e)
        _check(R, root, first, 4096)
        _check(R, root, first + (1 << 23) - 4096, 4096)
