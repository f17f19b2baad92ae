"""A call whose launch would need 2^32 threads or more in one dimension is refused: the runtime
takes such a grid with its size wrapped and runs a part of it.  Without a GPU only (the arguments
are no device memory; nothing may be launched with them).
"""
import ctypes as C

import pytest
import torch

from paper_2404_04270_amd import binding as B

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="passes made-up addresses")
SS_ERR_UNSUPPORTED = 2


@pytest.mark.parametrize("Bcap,refused", [(1 << 26, True), ((1 << 26) - 4, False)])
def test_lookup_of_2_to_the_32_threads(Bcap, refused):
    tables = B._CTables(1, 256, 1000, 1 << 20, None)
    rc = B._lib.ss_embbag_forward(C.byref(tables), C.c_void_p(1 << 20), C.c_int32(Bcap),
                                  C.c_int32(8), None, C.c_void_p(1 << 20), None)
    assert rc != 0 and ("grid too large" in B.ss_last_error()) == refused
    assert (rc == SS_ERR_UNSUPPORTED) == refused
