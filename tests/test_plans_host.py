"""Host only: the plans of dense and gathered-rows attention, made for an MI355X (the device that
plans are made for where none is visible)."""
import ctypes

import pytest

import paper_2408_07092_amd as ds


class DensePlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("units", "G", "ch", "n_ch")] + \
               [(n, ctypes.c_size_t) for n in ("off_ctl", "off_part", "total")]


def dense_plan(units, G, n_tokens, workspace_bytes=2 ** 64 - 1):
    """make_dense_plan of the library (an internal C++ function: by its mangled name)."""
    fn = getattr(ds.lib(), "_ZN2ds15make_dense_planERK10ds_shape_tiPNS_9DensePlanEm")
    fn.restype = ctypes.c_bool
    fn.argtypes = [ctypes.POINTER(ds.binding.DsShape), ctypes.c_int, ctypes.POINTER(DensePlan), ctypes.c_size_t]
    plan = DensePlan()
    shp = ds.shape(1, units * G, units, 128, n_tokens, n_tokens, 8, 1)
    assert fn(ctypes.byref(shp), n_tokens, ctypes.byref(plan), workspace_bytes)
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


@pytest.mark.parametrize("units", [1, 3, 12, 32, 200, 512])
@pytest.mark.parametrize("G", [1, 2, 7, 16, 64])
@pytest.mark.parametrize("k", [0, 1])
def test_workspace_for_more_tokens_serves_fewer(units, G, k):
    """A workspace of ds_workspace_bytes() for some number of tokens is enough for dense decode of
    every smaller number (a cache that grows by a token per step is one allocation)."""
    lengths = [1, 33, 100, 256, 300, 512, 600, 800, 1024, 1300, 2048, 4096, 5000, 8191, 8192, 16384, 40000, 65536]
    for i, longer in enumerate(lengths):
        have = ds.ds_workspace_bytes(ds.shape(1, units * G, units, 128, longer, longer, 8, k * max(1, longer // 16)))
        for tokens in lengths[:i + 1]:
            p = dense_plan(units, G, tokens, have)
            assert p.total <= have, (tokens, longer, p.n_ch)
            assert p.off_part + units * G * p.n_ch * 132 * 4 <= p.total
