"""Host only: the plans of dense and gathered-rows attention, made for an MI355X (the device that
plans are made for where none is visible)."""
import ctypes

import pytest

import paper_2408_07092_amd as ds


class DensePlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("units", "G", "ch", "n_ch")] + \
               [(n, ctypes.c_size_t) for n in ("off_ctl", "off_part", "total")]


def dense_plan(units, G, n_tokens):
    """make_dense_plan of the library (an internal C++ function: by its mangled name)."""
    fn = getattr(ds.lib(), "_ZN2ds15make_dense_planERK10ds_shape_tiPNS_9DensePlanE")
    fn.restype = ctypes.c_bool
    fn.argtypes = [ctypes.POINTER(ds.binding.DsShape), ctypes.c_int, ctypes.POINTER(DensePlan)]
    plan = DensePlan()
    shp = ds.shape(1, units * G, units, 128, n_tokens, n_tokens, 8, 1)
    assert fn(ctypes.byref(shp), n_tokens, ctypes.byref(plan))
    return plan


@pytest.fixture(autouse=True)
def mi355x():
    ds.ds_pretend_device(256, 8, 160 << 10)
    yield
    ds.ds_pretend_device(0, 0, 0)


# (units, heads per unit, tokens, chunk counts within 10 % of the fastest of those measured on an MI355X)
@pytest.mark.parametrize("units,G,tokens,lo,hi", [
    (1, 64, 2048, 6, 10),      # 8: 50.4 us, 32: 76.8, 64: 123
    (2, 64, 1024, 4, 10),
    (1, 64, 256, 1, 1),        # one chunk 28.1 us, 4: 36.2, 8: 40.5
    (1, 16, 2048, 6, 10),      # 8: 14.9 us, 32: 21.1, 64: 33.1
    (1, 8, 2048, 8, 16),
    (4, 8, 512, 4, 8),
    (1, 4, 2048, 12, 32),
    (1, 1, 2048, 24, 48),      # 32: 6.2 us, 64: 6.8
    (64, 1, 512, 4, 11),
    (48, 1, 1024, 8, 16),
    (32, 1, 65536, 8, 16),     # 8: 152 us, 64: 180
    (64, 1, 65536, 4, 8),
    (32, 4, 32768, 8, 16),
    (8, 8, 32768, 28, 36),     # 32: 31.9 us, 128: 69.5
    (12, 8, 20000, 18, 24),
    (512, 1, 4096, 1, 5),
])
def test_dense_plan_takes_a_chunk_count_near_the_fastest(units, G, tokens, lo, hi):
    p = dense_plan(units, G, tokens)
    assert lo <= p.n_ch <= hi and (p.n_ch - 1) * p.ch < tokens <= p.n_ch * p.ch and p.ch % 16 == 0
