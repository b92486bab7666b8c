"""The limit of tiles of the batch without a plan, for a call without a launch shape: in tiles of
128 points, refused before anything is launched, whichever kernel the call would run."""
import ctypes

import pytest

from paper_1804_10120_amd import _abi
from paper_1804_10120_amd._abi import CField, Domain, Field

LIMIT = 128 * _abi.TL_NOALLOC_MAX_TILES


def domains(sizes):
    """Subgrids at addresses that are never dereferenced, one after the other."""
    arr, at = (Domain * len(sizes))(), 1 << 40

    def take(ncomp, n, kind):
        nonlocal at
        f = kind(at, n)
        at += ncomp * n * 8
        return f
    for i, n in enumerate(sizes):
        arr[i] = Domain(n, *[take(c, n, CField) for c in (6, 18, 3, 9, 6, 1)], take(6, n, Field))
    return arr


@pytest.mark.parametrize("sizes", [[LIMIT // 2, LIMIT // 2 + 1], [LIMIT + 1],
                                   [1 << 20] * 32 + [1]],
                         ids=["two", "one_of_4_GiB", "many"])
def test_default_beyond_the_limit_of_tiles(sizes):
    """Two subgrids and many come with the descriptors in the arguments; one has a field of more
    than 4 GiB and would write the tables."""
    L = _abi.lib()
    assert L.tl_batch_run_noalloc(domains(sizes), len(sizes), None, None) == _abi.TL_ERR_SIZE
    assert b"tiles of 128 points" in ctypes.c_char_p(L.tl_last_error()).value
