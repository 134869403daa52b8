"""The screening's workspace: its size over all satellite counts, and the sizes the
no-allocation call takes, which end where the workspace passes its 64 MiB.

The size is the device-memory path's: a 256-byte header, bucket offsets for n / 4
buckets (16 at least, 2^20 at most) and an end, eight and four bytes a point, the
first three parts padded to 256 bytes.  The column path fits into it wherever it
is taken.
"""
import pytest

from paper_2603_27830_amd import _native


def expected(n, T):
    pad = lambda x: (x + 255) // 256 * 256  # noqa: E731
    buckets = min(max(n // 4, 16), 1 << 20)
    return 256 + pad(T * (buckets + 1) * 4) + pad(8 * n * T) + 4 * n * T


@pytest.mark.parametrize("n", [2, 63, 64, 3073, 12289, 199_999, 200_000, 200_001, 4_194_303, 4_194_304, 4_194_308,
                               5_200_001, 7_000_000])
@pytest.mark.parametrize("T", [1, 3, 64, 1000])
def test_size(n, T):
    assert _native.lib().sgp4_screen_workspace_bytes(n, T) == expected(n, T)


@pytest.mark.parametrize("n,T", [(9341, 551), (200_000, 25), (200_001, 25), (5_162_300, 1), (5_242_000, 1), (5_243_000, 1)])
def test_no_allocation_call_takes_what_fits(n, T):
    # the size (-2) is checked before the pointers (-1), so no device memory is touched
    rc = _native.lib().sgp4_screen_noalloc(None, _native.SGP4_FP64, None, n, T, 10.0, 0, None, None, None, None)
    fits = expected(n, T) <= 64 << 20
    assert rc == (-1 if fits else -2)
