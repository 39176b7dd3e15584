"""Host only: the plans of dense and gathered-rows attention and of the 4-bit label build, made for an
MI355X (the device that plans are made for where none is visible)."""
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


class Q4Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("launches", "tile", "n_wg", "per_wg", "n_max")]


def q4_plan(units, L, r):
    fn = getattr(ds.lib(), "_ZN2ds12make_q4_planERK10ds_shape_tPNS_6Q4PlanE")
    fn.restype, fn.argtypes = None, [ctypes.POINTER(ds.binding.DsShape), ctypes.POINTER(Q4Plan)]
    plan = Q4Plan()
    fn(ctypes.byref(ds.shape(1, units, units, 128, L, L, r, 1)), ctypes.byref(plan))
    return plan


@pytest.mark.parametrize("cus", [256, 64, 8])
@pytest.mark.parametrize("r", [1, 5, 8, 16, 24, 40, 64, 100, 128])
def test_q4_build_waits_only_for_workgroups_that_the_device_holds(cus, r):
    """Workgroups of the 4-bit label build wait for each other only where each die holds four units'
    shares at once; a tile fits the LDS that a launch gets without asking for more, up to the longest
    cache that the card's memory holds (1.1e9 rows of K); and the tiles cover the tokens."""
    ds.ds_pretend_device(cus, 8, 160 << 10)
    words = (r + 7) // 8
    seen = set()
    for units in (1, 3, 4, 32, 256, 5000):
        for L in (1, 7, 64, 65, 300, 1024, 1025, 5000, 16384, 65536, 131073, 262144, 1 << 20, 8400000, 1 << 24, 1100000000):
            p = q4_plan(units, L, r)
            seen.add(p.launches)
            lds = p.tile * 16 * words
            assert lds <= 60 << 10 and (p.n_wg - 1) * p.tile < L <= p.n_wg * p.tile
            assert p.n_wg * 256 < 1 << 32
            if p.launches == 1:
                assert p.n_wg == 1
            elif p.launches == 2:
                held = min(8, (160 << 10) // (lds + 1280)) * (cus // 8)
                assert 1 < p.n_wg <= 128 and 4 * -(-p.n_wg // 8) <= held
            else:
                assert p.launches == 3 and (p.n_max - 1) * p.per_wg < L <= p.n_max * p.per_wg
    assert seen == ({1, 2, 3} if cus > 8 or r >= 64 else seen | {1, 3})


@pytest.mark.parametrize("units,G,tokens,r,kind,one", [
    (32, 1, 6144, 8, 0, True), (32, 1, 6145, 8, 0, False), (32, 1, 6144, 16, 0, True), (32, 1, 6144, 24, 0, True),
    (128, 1, 8192, 24, 0, True), (128, 1, 8193, 8, 0, False), (127, 1, 8192, 8, 0, False), (64, 1, 6144, 16, 2, True),
    (32, 4, 6144, 8, 0, True), (32, 4, 6145, 8, 0, False), (32, 4, 6144, 12, 0, True), (32, 4, 6144, 8, 2, True),
    (32, 4, 5376, 16, 0, True), (32, 4, 5377, 16, 0, False), (8, 8, 6000, 16, 2, False), (8, 8, 6000, 12, 2, False),
    (128, 4, 8192, 8, 0, True), (128, 4, 6656, 24, 0, True), (128, 4, 6657, 24, 0, False), (128, 4, 8192, 12, 0, True),
    (128, 8, 6657, 16, 2, False), (128, 2, 6144, 8, 0, True), (128, 2, 6145, 8, 0, False), (128, 2, 5632, 16, 2, True),
    (128, 2, 5633, 16, 2, False), (64, 2, 5000, 8, 0, False),
])
def test_one_workgroup_per_unit_up_to_a_line(units, G, tokens, r, kind, one):
    """Both sides of the rule for units of 4K to 8K tokens, and of its limit of a sixteenth in rows."""
    wgs = lambda k: ds.ds_plan_describe(ds.shape(1, units * G, units, 128, tokens, (tokens + 3) // 4 * 4, r, k),
                                        kind)["workgroups_per_unit"]
    assert (wgs(tokens // 16) == 1) == one
    if one:
        half = 2 * units >= 256
        wide = r > (8 if kind == 2 else 12)
        line = (8192 if half else 6144) if G == 1 else (5632 if wide else 6144) if G == 2 else \
               (6656 if wide else 8192) if half else (5376 if wide else 6144)
        assert wgs(line // 16) == 1 and wgs(line // 16 + 1) > 1


def smallest_workspace(shp):
    """Bytes from which ds_sparse_decode no longer refuses the workspace: host only, a misaligned K is
    refused after it and before anything is enqueued."""
    fake, bad = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x10010)
    status = lambda n: ds.lib().ds_sparse_decode(fake, fake, bad, fake, fake, fake, None, fake, n, ctypes.byref(shp), None)
    lo, hi = 0, ds.ds_workspace_bytes(shp)
    assert status(hi) == ds.DS_ERR_ALIGN and status(lo) == ds.DS_ERR_WORKSPACE
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if status(mid) == ds.DS_ERR_WORKSPACE:
            lo = mid
        else:
            hi = mid
    return hi


@pytest.mark.parametrize("r", [4, 12, 20, 24, 28, 32])
@pytest.mark.parametrize("units,G,L", [(2, 1, 3000), (12, 7, 20011), (32, 1, 65536), (128, 2, 9000), (1, 1, 262144)])
def test_scoring_in_the_attention_launch_needs_no_larger_workspace(units, G, L, r):
    """Label widths that may be scored in the attention launch ask for no more than the plan with a
    scoring launch does."""
    shp = ds.shape(1, units * G, units, 128, L, L, r, L // 16)
    need = smallest_workspace(shp)
    ds.ds_tune_set(4, 1)
    try:
        assert smallest_workspace(shp) == need
    finally:
        ds.ds_tune_set(4, 0)


def test_label_widths_that_the_attention_launch_scores():
    """Every multiple of 4 up to 32, and no other."""
    for r in range(1, 129):
        si = ds.ds_plan_describe(ds.shape(1, 32, 32, 128, 4096, 4096, r, 256))["scores_itself"]
        assert si == (r % 4 == 0 and r <= 32), r


@pytest.mark.parametrize("units,G,L,chunk", [
    (16, 1, 65536, 1024), (17, 1, 65536, 2048), (20, 2, 65536, 2048), (48, 1, 32768, 2048), (8, 1, 131072, 1024),
    (9, 1, 131072, 2048), (40, 1, 16384, 1024), (32, 1, 65536, 2048), (40, 1, 65536, 4096), (150, 2, 9000, 2048),
])
def test_chunks_behind_a_scoring_launch_fit_at_once(units, G, L, chunk):
    """Single heads and pairs that a separate launch scores: four workgroups to a compute unit, as many
    as the kernel's registers allow, and not a second round for a few more."""
    for kind, r in ((1, 8), (0, 64), (0, 7), (2, 32)):
        p = ds.ds_plan_describe(ds.shape(1, units * G, units, 128, L, L, r, L // 16), kind)
        assert p["scores_itself"] == 0 and p["tokens_per_workgroup"] == chunk
        assert p["workgroups"] <= 4 * 256 or chunk == 4096


@pytest.mark.parametrize("units,G,L,r,lo,hi", [
    # (units, heads per unit, tokens, channels, workgroups per unit within a few percent of the fastest measured)
    (32, 1, 65536, 8, 7, 8), (32, 1, 262144, 8, 16, 16), (128, 1, 32768, 8, 4, 4), (64, 1, 16384, 8, 4, 4),
    (32, 1, 16384, 8, 6, 8), (32, 1, 8192, 8, 3, 6), (1, 1, 262144, 8, 25, 64), (96, 1, 30000, 8, 4, 5),
    (12, 7, 20011, 12, 6, 12), (8, 8, 131072, 8, 14, 26), (128, 8, 32768, 8, 2, 4), (32, 8, 65536, 8, 8, 16),
    # one workgroup per unit, or several
    (192, 4, 9000, 8, 1, 1), (192, 8, 16384, 16, 1, 1), (191, 4, 9000, 8, 2, 4), (192, 4, 16385, 8, 2, 4),
    (192, 1, 16384, 8, 1, 1), (192, 1, 16385, 8, 2, 4), (1024, 8, 12000, 8, 1, 1),
])
def test_chunks_of_a_launch_that_scores_itself(units, G, L, r, lo, hi):
    """Workgroups per unit of the decode launch; several of them are resident at once, and none has
    more than 16384 tokens."""
    p = ds.ds_plan_describe(ds.shape(1, units * G, units, 128, L, L, r, L // 16))
    n, ch, launches = p["workgroups_per_unit"], p["tokens_per_workgroup"], p["launches_planned"]
    assert p["scores_itself"] == 1 and lo <= n <= hi and ch <= 16384 and (n - 1) * ch < L <= n * ch
    assert n == 1 or -(-units // launches) * n <= 2 * 256


@pytest.mark.parametrize("units,G,L,r,kind", [
    (32, 1, 65536, 8, 0), (12, 7, 20011, 12, 0), (5, 16, 40000, 32, 0), (300, 2, 20000, 4, 0), (700, 4, 20000, 8, 2),
    (1, 1, 1000000, 8, 0), (2, 33, 100000, 16, 2), (200, 1, 100000, 24, 0),
])
def test_decode_plans_of_every_device_size_are_within_bounds(units, G, L, r, kind):
    """On devices of 8 to 256 compute units: chunks cover the tokens, fit the kernels, and are no more
    than the workspace has partials for."""
    for cus in (8, 64, 120, 256):
        ds.ds_pretend_device(cus, 8, 160 << 10)
        shp = ds.shape(1, units * G, units, 128, L, (L + 3) // 4 * 4, r, L // 16)
        p = ds.ds_plan_describe(shp, kind)
        n, ch = p["workgroups_per_unit"], p["tokens_per_workgroup"]
        assert (n - 1) * ch < L <= n * ch and ch % 4 == 0
        prefix = units * (64 + 4096 * 4 + 256 * 4 + 4 * ((L + 3) // 4) * 4 + 8 * L)
        assert prefix + units * G * n * 132 * 4 <= ds.ds_workspace_bytes(shp)
        if p["scores_itself"]:
            assert ch <= 16384 and p["launches_planned"] <= 3
            per_cu = 1 if cus < 128 else 3 if G > 8 else 2
            assert n == 1 or -(-units // p["launches_planned"]) * n <= per_cu * cus
