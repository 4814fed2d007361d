"""Copies between ciphertexts and host memory: pageable buffers of several
chunks (with a remainder), unaligned ones, and pinned ones."""
import ctypes as C

import numpy as np
import pytest

from paper_2305_17341_amd import he, inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chain,level", [(I.TOY, 0), (I.SMALL, 3), (I.SMALL, 1), (I.SERVE15, 14), (I.SERVE15, 6)],
                         ids=lambda v: getattr(v, "name", v))
def test_export_and_import_return_the_words(chain, level):
    ctx = he.chain_context(chain, seed=3)
    lib = he.load()
    words = 2 * (level + 1) * ctx.N
    rng = I.rng(17)
    moduli = ctx.moduli[:level + 1]
    want = np.concatenate([rng.integers(0, q, ctx.N, dtype=np.uint64) for q in list(moduli) * 2])
    odd = np.empty(words * 8 + 8, dtype=np.uint8)[3:3 + words * 8]  # a host address that is no multiple of 8
    odd[:] = want.view(np.uint8)
    pin = C.c_void_p()
    assert lib.hipHostMalloc(C.byref(pin), C.c_size_t(words * 8), C.c_uint(0)) == 0
    pinned = np.ctypeslib.as_array(C.cast(pin, he.u64p), (words,))
    handles = []
    for src in (want.ctypes.data, odd.ctypes.data):
        h = C.c_void_p()
        assert lib.he_ct_import(ctx.ptr, C.cast(src, he.u64p), words, level, 2.0 ** 40, C.byref(h)) == 0
        handles.append(h)
        src_done = np.array(want)
        back = np.zeros(words, dtype=np.uint64)
        odd_back = np.zeros(words * 8 + 8, dtype=np.uint8)[5:5 + words * 8]
        pinned[:] = 0
        for dst in (back.ctypes.data, odd_back.ctypes.data, pin.value):
            assert lib.he_ct_export(h, C.cast(dst, he.u64p), words, None, None) == 0
        np.testing.assert_array_equal(back, src_done)
        np.testing.assert_array_equal(odd_back, src_done.view(np.uint8))
        np.testing.assert_array_equal(pinned, src_done)
    for h in handles:
        lib.he_ct_free(h)
    assert lib.hipHostFree(pin) == 0
