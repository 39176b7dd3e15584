"""GPU checks of single kernels at the sizes where a tile, a remainder or a dispatch rule can go
wrong, against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2408_07092_amd as ds
from oracle import ds_oracle as O
from tests.parity_util import Case, check_output, full_parity, to_dev
from tests.test_plans_host import q4_plan, smallest_workspace
from workloads import Workload, make_layer_numpy, make_layer_torch

pytestmark = pytest.mark.gpu


def rand_channels(Hkv, r, seed):
    rng = np.random.default_rng(seed)
    return np.stack([np.sort(rng.permutation(128)[:r]) for _ in range(Hkv)]).astype(np.int32)


def launches_of(fn):
    """{kernel: launches} of the library's kernels that `fn` enqueues."""
    ds.ds_profile_reset()
    ds.ds_profile_enable(True)
    try:
        fn()
        torch.cuda.synchronize()
        return {name: n for name, (_, n) in ds.ds_profile_read().items()}
    finally:
        ds.ds_profile_enable(False)
        ds.ds_profile_reset()


ALONE, WAITS, TWO_READS = ["k_q4_build"], ["k_q4_build", "waits"], ["k_q4_amax", "k_q4_code"]


@pytest.mark.parametrize("B,Hkv,L,L_max,r,spin,plan", [
    (1, 1, 1, 1, 1, 0, ALONE),               # one token
    (2, 3, 64, 64, 8, 0, ALONE),
    (1, 2, 65, 70, 3, 0, ALONE),
    (1, 3, 64, 64, 128, 0, ALONE),           # the longest unit that one workgroup takes: every channel ...
    (1, 3, 65, 66, 128, 0, TWO_READS),       # ... and one token more
    (1, 2, 1024, 1024, 8, 0, ALONE),         # ... of 8 channels ...
    (1, 2, 1025, 1028, 8, 0, TWO_READS),
    (1, 2, 1025, 1028, 16, 0, TWO_READS),
    (8, 32, 1290, 1290, 20, 0, WAITS),       # units that fill the device, one tile too long for one workgroup
    (8, 32, 1280, 1281, 20, 0, ALONE),       # ... and just not (60 KiB of LDS)
    (1, 1, 40001, 40001, 8, 0, TWO_READS),   # few units wait for nobody
    (1, 2, 700, 700, 128, 0, TWO_READS),
    (1, 2, 3000, 3000, 100, 0, TWO_READS),   # idle threads in a pass
    (4, 1, 2047, 2047, 8, 0, TWO_READS),     # the least work for a wait ...
    (4, 1, 2048, 2050, 8, 0, WAITS),
    (4, 3, 4100, 4100, 12, 0, WAITS),        # ... of two words a token, idle threads
    (2, 12, 2049, 2049, 100, 0, TWO_READS),  # 64 channels and more: four rounds to a tile
    (5, 10, 1250, 1251, 128, 0, WAITS),      # 16 words a token, workgroups of 50 tokens
    (1, 32, 6250, 6250, 64, 0, WAITS),
    (4, 1, 270000, 270000, 8, 0, WAITS),     # a hundred workgroups per unit
    (4, 1, 530000, 530000, 8, 0, TWO_READS), # more than 128 would have to wait
    (2, 4, 9000, 9000, 12, 1, WAITS),        # waits that run out: a workgroup finds the maxima by itself
    (1, 8, 2500, 2500, 8, 1, WAITS),
])
def test_q4_build_tiles(B, Hkv, L, L_max, r, spin, plan):
    """Codes and maxima bit-equal to the oracle's on both sides of the rules that choose between one
    workgroup per unit, workgroups that wait and two reads, and when a workgroup stops waiting for the
    others of its unit."""
    w = Workload("t", B, Hkv, Hkv, 128, L, r, 1, 1)
    t = make_layer_numpy(w, L_max=L_max)
    ch = rand_channels(Hkv, r, seed=L + r)
    W = (r + 7) // 8
    codes = torch.full((B, Hkv, L_max, W), -1, dtype=torch.int32, device="cuda")
    amax = torch.full((B, Hkv, r), -1.0, dtype=torch.float32, device="cuda")
    shp = ds.shape(B, Hkv, Hkv, 128, L, L_max, r, 1)
    K, chd = to_dev(t["K"]), to_dev(ch)
    ds.ds_tune_set(5, spin)
    try:
        ran = launches_of(lambda: ds.ds_build_label_q4(K, chd, codes, amax, shp))
    finally:
        ds.ds_tune_set(5, 0)
    assert sorted(ran) == [k for k in plan if k.startswith("k_")]
    assert (q4_plan(B * Hkv, L, r).n_wg > 1) == (plan is not ALONE)
    want_codes, want_amax = O.build_label_q4(t["K"], ch, L)
    assert np.array_equal(amax.cpu().numpy(), want_amax)
    assert np.array_equal(codes.cpu().numpy()[:, :, :L].view(np.uint32), want_codes[:, :, :L])
    assert (codes[:, :, L:] == -1).all()


def test_q4_build_on_a_device_that_holds_few_workgroups():
    """Told of a device of 8 compute units, the build has no workgroup wait for more than the device
    holds four times over; the codes are the same."""
    B, Hkv, L, r = 2, 4, 20000, 16
    w = Workload("t", B, Hkv, Hkv, 128, L, r, 1, 1)
    t = make_layer_numpy(w)
    ch = rand_channels(Hkv, r, seed=1)
    K, chd = to_dev(t["K"]), to_dev(ch)
    codes = torch.empty((B, Hkv, L, 2), dtype=torch.int32, device="cuda")
    amax = torch.empty((B, Hkv, r), dtype=torch.float32, device="cuda")
    build = lambda: ds.ds_build_label_q4(K, chd, codes, amax, ds.shape(B, Hkv, Hkv, 128, L, L, r, 1))
    assert list(launches_of(build)) == ["k_q4_build"]
    ds.ds_pretend_device(8, 8, 160 << 10)
    try:
        codes.fill_(-1)
        assert sorted(launches_of(build)) == TWO_READS
    finally:
        ds.ds_pretend_device(0, 0, 0)
    want_codes, want_amax = O.build_label_q4(t["K"], ch, L)
    assert np.array_equal(amax.cpu().numpy(), want_amax)
    assert np.array_equal(codes.cpu().numpy().view(np.uint32), want_codes)


@pytest.mark.parametrize("B,Hkv,L,r,plan", [(2, 4, 300, 16, ALONE), (2, 4, 20000, 16, WAITS), (1, 2, 5000, 24, TWO_READS)])
def test_q4_build_on_streams_and_in_a_graph(B, Hkv, L, r, plan):
    """Three streams that build at the same time, and a captured build that is replayed with other K
    rows: the oracle's codes and maxima each time."""
    shp = ds.shape(B, Hkv, Hkv, 128, L, L, r, 1)
    assert q4_plan(B * Hkv, L, r).launches == {"k_q4_amax": 3}.get(plan[0], len(plan))
    ch = rand_channels(Hkv, r, seed=L)
    chd = to_dev(ch)
    sets = []
    for i in range(3):
        K = make_layer_numpy(Workload("t", B, Hkv, Hkv, 128, L, r, 1, 1), layer=i)["K"]
        sets.append((K, to_dev(K), torch.empty((B, Hkv, L, (r + 7) // 8), dtype=torch.int32, device="cuda"),
                     torch.empty((B, Hkv, r), dtype=torch.float32, device="cuda"), O.build_label_q4(K, ch, L)))

    def check(codes, amax, want):
        assert np.array_equal(amax.cpu().numpy(), want[1])
        assert np.array_equal(codes.cpu().numpy().view(np.uint32), want[0])

    streams = [torch.cuda.Stream() for _ in sets]
    torch.cuda.synchronize()
    for _ in range(5):
        for st, (_, K, codes, amax, _) in zip(streams, sets):
            ds.ds_build_label_q4(K, chd, codes, amax, shp, stream=st)
    torch.cuda.synchronize()
    for _, _, codes, amax, want in sets:
        check(codes, amax, want)
    Kg, codes, amax = sets[0][1].clone(), torch.empty_like(sets[0][2]), torch.empty_like(sets[0][3])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds.ds_build_label_q4(Kg, chd, codes, amax, shp)
    for _, K, _, _, want in sets + sets[:1]:
        Kg.copy_(K)
        codes.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        check(codes, amax, want)


@pytest.mark.parametrize("B,Hkv,L,L_max,r,kv", [
    (1, 1, 1, 1, 1, False),          # one token, one channel
    (1, 1, 2, 5, 128, False),        # one pass of two rows
    (2, 3, 300, 301, 24, False),     # equal shares, idle threads in a pass
    (1, 2, 33, 33, 100, True),       # interleaved rows, a remainder in the last pass
    (3, 40, 1700, 1700, 8, False),   # 50 MiB: more workgroups per compute unit ...
    (4, 32, 3300, 3301, 16, False),  # ... 103 MiB: and more
    (8, 16, 6400, 6400, 24, False),  # the first size with the streaming mark and eight passes in flight (200 MiB)
    (4, 16, 6401, 6401, 7, True),    # ... of interleaved rows, idle threads and a remainder
    (8, 16, 6400, 6400, 64, False),  # 64 channels: one pass at a time at every size
])
def test_label_build_sizes(B, Hkv, L, L_max, r, kv):
    """Bit copies on both sides of the rules that choose the rows of a workgroup and the streaming mark."""
    g = torch.Generator(device="cuda").manual_seed(L + r)
    rows = 2 if kv else 1
    K = torch.randint(-32768, 32768, (B, Hkv, L_max, rows, 128), dtype=torch.int16, device="cuda", generator=g)
    ch = to_dev(rand_channels(Hkv, r, seed=L + r))
    label = torch.full((B, Hkv, L_max, r), 0x7e01, dtype=torch.int16, device="cuda")
    shp = ds.shape(B, Hkv, Hkv, 128, L, L_max, r, 1)
    (ds.ds_build_label_kv if kv else ds.ds_build_label)(K, ch, label, shp)
    torch.cuda.synchronize()
    want = torch.gather(K[:, :, :L, 0], 3, ch.long()[None, :, None, :].expand(B, Hkv, L, r))
    assert torch.equal(label[:, :, :L], want)
    assert (label[:, :, L:] == 0x7e01).all()


@pytest.mark.parametrize("B,Hq,Hkv,L,L_max", [
    (1, 1, 1, 1, 1),
    (1, 1, 1, 33, 40),           # one row more than the smallest chunk of a device full of chunks
    (1, 8, 1, 4099, 4100),       # one unit in groups of 8: many chunks, a ragged last one
    (3, 28, 4, 2003, 2048),      # groups of 7
    (2, 40, 40, 700, 700),       # single heads, several workgroups per compute unit
    (9, 64, 32, 130, 130),       # more units than compute units, pairs
    (5, 64, 64, 65, 65),         # the same, single heads
    (1, 32, 1, 1000, 1000),      # groups of 32: two passes over the rows
])
def test_dense_decode_chunk_rule(B, Hq, Hkv, L, L_max):
    """Dense decode at both ends of the rule that cuts a unit into chunks."""
    w = Workload("t", B, Hq, Hkv, 128, L, 8, 1, 1)
    t = make_layer_numpy(w, L_max=L_max)
    shp = ds.shape(B, Hq, Hkv, 128, L, L_max, 8, 1)
    ws = ds.ds_workspace_alloc(shp)
    out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ds.ds_dense_decode(to_dev(t["q"]), to_dev(t["K"]), to_dev(t["V"]), out, ws, shp)
    torch.cuda.synchronize()
    check_output(out.cpu().numpy(), O.dense_decode(t["q"], t["K"], t["V"], L), f"dense {(B, Hq, Hkv, L)}")


@pytest.mark.parametrize("Hq,Hkv,L", [
    (64, 1, 300),                # one chunk, four passes over the rows
    (64, 1, 2048),               # several chunks, eight rounds of heads in the merge
    (34, 2, 1000),               # groups of 17: a second pass with one head
    (2, 1, 2000),                # pairs: chunks of whole rounds
])
def test_dense_decode_chunk_rule_of_large_groups(Hq, Hkv, L):
    test_dense_decode_chunk_rule(1, Hq, Hkv, L, L)


@pytest.mark.parametrize("Hq,Hkv,L,L_ws", [(1, 1, 256, 300), (1, 1, 1024, 1300), (4, 1, 800, 1300), (56, 8, 800, 800)])
def test_dense_decode_in_the_workspace_of_more_tokens(Hq, Hkv, L, L_ws):
    """A workspace sized for more tokens (or one with room for chunks of 64 tokens and no more) is not
    refused where the chunk rule would like a larger one: fewer chunks, the same result."""
    w = Workload("t", 1, Hq, Hkv, 128, L, 8, 1, 1)
    t = make_layer_numpy(w)
    shp = ds.shape(1, Hq, Hkv, 128, L, L, 8, 0)
    n = ds.ds_workspace_bytes(ds.shape(1, Hq, Hkv, 128, L_ws, L_ws, 8, 0))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    ds.ds_workspace_init(ws)
    out = torch.full((1, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ds.ds_dense_decode(to_dev(t["q"]), to_dev(t["K"]), to_dev(t["V"]), out, ws, shp)
    torch.cuda.synchronize()
    check_output(out.cpu().numpy(), O.dense_decode(t["q"], t["K"], t["V"], L), f"dense {(Hq, Hkv, L, L_ws)}")


@pytest.mark.parametrize("B,Dm,N", [(1, 8, 5), (1, 512, 4), (3, 520, 1025), (5, 4096, 65), (1, 4104, 33), (2, 8192, 4100),
                                    # one past each number of pieces in flight, read once with and without
                                    # the streaming mark (64 MiB of Wq) and once per four rows of a batch
                                    (4, 1032, 9), (9, 2056, 40), (4, 512, 65537), (17, 512, 65537), (1, 4096, 8192),
                                    (6, 4096, 8193), (4, 8192, 4096), (7, 8184, 4100)])
def test_predict_query_pieces(B, Dm, N):
    """Row lengths at the edges of the pieces in flight and feature counts at the edges of the
    workgroups: one fp16 step plus the binary32 error of Dm products from the float64 oracle."""
    rng = np.random.default_rng(Dm + N)
    x = rng.standard_normal((B, Dm)).astype(np.float16)
    Wq = (rng.standard_normal((N, Dm)) / np.sqrt(Dm)).astype(np.float16)
    q = torch.full((B, N), float("nan"), dtype=torch.float16, device="cuda")
    ds.ds_predict_query(to_dev(x), to_dev(Wq), q)
    torch.cuda.synchronize()
    got, ref = q.cpu().numpy().astype(np.float64), O.predict_query(x, Wq).astype(np.float64)
    mag = np.abs(x.astype(np.float64)) @ np.abs(Wq.astype(np.float64)).T
    step = np.maximum(np.spacing(np.abs(ref).astype(np.float16)).astype(np.float64), 2.0 ** -24)
    assert (np.abs(got - ref) <= step + Dm * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("B,Hkv,L,k", [(1, 1, 5, 1), (1, 3, 40, 33), (2, 4, 700, 97), (1, 2, 3000, 1600),
                                        (1, 8, 64, 64), (1, 1, 600, 513), (3, 19, 9, 9), (1, 1, 900, 512)])
def test_gather_rows_host_rounds(B, Hkv, L, k):
    """Row counts below, at and beyond one round of the gather's workgroups, with unused entries."""
    rng = np.random.default_rng(k)
    K = torch.from_numpy(rng.standard_normal((B, Hkv, L, 128)).astype(np.float16)).pin_memory()
    V = torch.from_numpy(rng.standard_normal((B, Hkv, L, 128)).astype(np.float16)).pin_memory()
    idx = rng.integers(0, L, size=(B, Hkv, k)).astype(np.int32)
    idx[rng.random(idx.shape) < 0.1] = -1
    rows = torch.full((B, Hkv, k, 2, 128), float("nan"), dtype=torch.float16, device="cuda")
    ds.ds_gather_rows_host(K, V, to_dev(idx), rows, ds.shape(B, Hkv, Hkv, 128, L, L, 8, k))
    torch.cuda.synchronize()
    take = np.maximum(idx, 0)[..., None].astype(np.int64)
    want = np.stack([np.take_along_axis(t.numpy(), take, axis=2) for t in (K, V)], axis=3)
    want[idx < 0] = 0
    assert np.array_equal(rows.cpu().numpy().view(np.uint16), want.view(np.uint16))


ONE, SEVERAL = True, False


@pytest.mark.parametrize("Hq,Hkv,L,L_max,r,k,cus,one,streams", [
    (1, 1, 1, 1, 4, 1, 0, ONE, False),              # one token
    (3, 3, 1500, 1501, 4, 93, 0, ONE, False),       # rows of 8 bytes, units on odd multiples of 8 bytes
    (2, 2, 9001, 9003, 4, 562, 0, SEVERAL, False),  # several workgroups per unit, a ragged last chunk
    (2, 1, 700, 701, 12, 50, 0, ONE, False),        # pairs, rows of three 8-byte pieces
    (7, 1, 9100, 9101, 12, 570, 0, SEVERAL, False), # groups of 7, several workgroups per unit
    (120, 120, 2100, 2100, 12, 131, 0, ONE, False), # many units that the caches hold
    (1, 1, 12000, 12000, 12, 750, 0, SEVERAL, False),  # single head, several workgroups
    (4, 4, 3000, 3001, 24, 187, 0, ONE, False),     # rows of three 16-byte pieces
    (16, 1, 8500, 8500, 24, 531, 0, SEVERAL, False),  # groups of 16
    (6, 6, 11000, 11000, 24, 300, 8, ONE, False),   # units enough for one workgroup of 1024 threads each
    (6, 6, 10950, 10951, 4, 300, 8, ONE, False),    # ... with 8-byte rows
    (6, 6, 16384, 16384, 12, 1024, 8, ONE, False),  # ... of the longest unit
    # calls that stream past the caches: single heads and pairs with one workgroup per unit and several
    (24, 24, 2500, 2500, 4, 1400, 0, ONE, True),
    (24, 24, 2500, 2501, 12, 1400, 0, ONE, True),
    (24, 24, 2500, 2500, 24, 1400, 0, ONE, True),
    (48, 24, 2500, 2501, 4, 1400, 0, ONE, True),
    (48, 24, 2500, 2500, 12, 1400, 0, ONE, True),
    (48, 24, 2500, 2500, 24, 1400, 0, ONE, True),
    (12, 12, 12000, 12001, 4, 2600, 0, SEVERAL, True),
    (12, 12, 12000, 12000, 12, 2600, 0, SEVERAL, True),
    (12, 12, 12000, 12000, 24, 2600, 0, SEVERAL, True),
    (24, 12, 12000, 12000, 4, 2600, 0, SEVERAL, True),
    (24, 12, 12000, 12001, 12, 2600, 0, SEVERAL, True),
    (24, 12, 12000, 12000, 24, 2600, 0, SEVERAL, True),
    # wider label rows: five and seven pieces of 8 bytes, four of 16
    (3, 3, 1500, 1501, 20, 93, 0, ONE, False),
    (2, 1, 9001, 9003, 20, 562, 0, SEVERAL, False),
    (12, 12, 12000, 12001, 20, 2600, 0, SEVERAL, True),
    (1, 1, 64, 65, 28, 9, 0, ONE, False),
    (48, 24, 2500, 2501, 28, 1400, 0, ONE, True),
    (6, 6, 10950, 10951, 28, 300, 8, ONE, False),
    (7, 1, 9100, 9101, 28, 570, 0, SEVERAL, False),
    (2, 2, 9001, 9003, 32, 562, 0, SEVERAL, False),
    (24, 24, 2500, 2501, 32, 1400, 0, ONE, True),
    (6, 6, 16384, 16384, 32, 1024, 8, ONE, False),
    (16, 1, 8500, 8500, 32, 531, 0, SEVERAL, False),
    (4, 1, 4000, 4001, 32, 250, 0, ONE, False),
    # both sides of the rule for units of 4K to 8K tokens
    (1, 1, 6144, 6144, 8, 384, 0, ONE, False),      # the longest unit that one workgroup takes of few units ...
    (1, 1, 6144, 6144, 8, 385, 0, SEVERAL, False),  # ... and a row more ...
    (4, 1, 6145, 6145, 8, 384, 0, SEVERAL, False),  # ... or a token more, in groups of 4
    (4, 1, 5376, 5376, 16, 336, 0, ONE, False),     # the same of wide label rows
    (4, 1, 5377, 5377, 16, 336, 0, SEVERAL, False),
    (4, 4, 8191, 8191, 8, 511, 8, ONE, False),      # units for half the device: one workgroup of 1024 threads each ...
    (4, 4, 8193, 8193, 8, 511, 8, SEVERAL, False),  # ... and several per unit
    (6, 3, 6100, 6100, 8, 380, 8, SEVERAL, False),  # pairs: several per unit ...
    (8, 4, 6100, 6100, 8, 380, 8, ONE, False),      # ... or one when there are units for half the device
    (8, 4, 6144, 6144, 8, 385, 8, SEVERAL, False),
])
def test_decode_label_rows_and_workgroups_per_unit(Hq, Hkv, L, L_max, r, k, cus, one, streams):
    """Label rows of every number of channels that the attention launch scores itself, and both
    sides of the rules that give a unit one workgroup (planned for a small device where they
    count units) and that mark loads as streaming (16 MiB of label and K/V rows)."""
    w = Workload("t", 1, Hq, Hkv, 128, L, r, k, 1)
    t = make_layer_numpy(w, L_max=L_max)
    assert (Hkv * (L * r * 2 + k * 512) >= 16 << 20) == streams
    if cus:
        ds.ds_pretend_device(cus, 8, 160 << 10)
    try:
        plan = ds.ds_plan_describe(ds.shape(1, Hq, Hkv, 128, L, L_max, r, k))
        assert plan["scores_itself"] == 1 and (plan["workgroups_per_unit"] == 1) == one
        case = Case(t["q"], t["K"], t["V"], rand_channels(Hkv, r, seed=L + r), L, k)
        full_parity(case, what=f"Hq{Hq} Hkv{Hkv} L{L} r{r} k{k}")
    finally:
        ds.ds_pretend_device(0, 0, 0)


@pytest.mark.parametrize("r", [12, 32])
def test_decode_in_the_smallest_workspace(r):
    """A workspace that holds the plan with a scoring launch and not the one without (planned for 16
    compute units, where the two differ): that plan, the same rows."""
    B, Hq, Hkv, L, k = 1, 12, 3, 33000, 4125
    shp = ds.shape(B, Hq, Hkv, 128, L, L, r, k)
    t = make_layer_numpy(Workload("t", B, Hq, Hkv, 128, L, r, k, 1))
    ch = rand_channels(Hkv, r, seed=r)
    q, K, V, chd = to_dev(t["q"]), to_dev(t["K"]), to_dev(t["V"]), to_dev(ch)
    label = torch.empty((B, Hkv, L, r), dtype=torch.float16, device="cuda")
    ds.ds_build_label(K, chd, label, shp)
    got = []
    ds.ds_pretend_device(16, 8, 160 << 10)
    try:
        for n in ((smallest_workspace(shp) + 15) // 16 * 16, ds.ds_workspace_bytes(shp)):
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            ds.ds_workspace_init(ws)
            out = torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda")
            idx = torch.full((B, Hkv, k), -1, dtype=torch.int32, device="cuda")
            ran = launches_of(lambda: ds.ds_sparse_decode(q, label, K, V, chd, out, idx, ws, shp))
            got.append(("k_score" in ran, idx.cpu().numpy(), out.cpu().numpy()))
    finally:
        ds.ds_pretend_device(0, 0, 0)
    assert got[0][0] and not got[1][0]
    assert np.array_equal(got[0][1], got[1][1])
    check_output(got[0][2], got[1][2].astype(np.float64), "smallest workspace")


@pytest.mark.parametrize("Hq,L,k,step,one", [
    (1, 12000, 800, 0.0, SEVERAL),      # every key the same: 12000 candidates, the tie cut among them all
    (2, 20000, 9000, 1e-3, SEVERAL),    # a few keys of many tokens each
    (4, 9000, 500, 1e-3, SEVERAL),      # matrix-core variant
    (1, 4000, 2900, 1e-3, ONE),         # one workgroup per unit
    (1, 5000, 3100, 1e-3, SEVERAL),
])
def test_decode_many_candidates(Hq, L, k, step, one):
    """Thousands of keys in the threshold bin, most of them equal: the whole workgroup settles the threshold, from
    lists that LDS does not hold; the index list is the oracle's, ties to the lowest token."""
    w = Workload("t", 1, Hq, 1, 128, L, 8, k, 1)
    t = make_layer_numpy(w)
    ch = rand_channels(1, 8, seed=L)
    t["q"][:] = np.float16(0.5)
    rng = np.random.default_rng(L)
    t["K"][0, 0][:, ch[0]] = (1.0 + step * rng.integers(0, 5, (L, 1))).astype(np.float16)
    assert (ds.ds_plan_describe(ds.shape(1, Hq, 1, 128, L, L, 8, k))["workgroups_per_unit"] == 1) == one
    case = Case(t["q"], t["K"], t["V"], ch, L, k)
    full_parity(case, what=f"many candidates L{L} k{k}")


@pytest.mark.parametrize("Hq,Hkv,L,r,k,cus,scores", [
    # scores far below and far above the label query's size: coarse bins
    (1, 1, 3000, 8, 187, 0, "tiny"), (2, 1, 12000, 16, 750, 0, "tiny"), (4, 1, 9000, 12, 563, 0, "tiny"),
    (1, 1, 3000, 8, 187, 0, "huge"), (3, 1, 9000, 8, 563, 0, "huge"), (1, 1, 12000, 4, 750, 0, "huge"),
    # thresholds on the negative side, and at either end of the list
    (1, 1, 4097, 8, 256, 0, "negative"), (2, 1, 9001, 8, 562, 0, "negative"), (8, 1, 20000, 8, 1250, 0, "negative"),
    (1, 1, 4096, 8, 2900, 0, "plain"), (1, 1, 20000, 8, 19999, 0, "plain"), (4, 1, 9000, 8, 1, 0, "plain"),
    # most tokens of a unit in one chunk of it
    (1, 1, 40000, 8, 2500, 0, "front"), (7, 1, 30000, 12, 1875, 0, "front"), (1, 1, 40000, 8, 20000, 0, "front"),
    # one workgroup of 16384 tokens, 32 keys to a thread: its edges (planned for eight compute units)
    (6, 6, 16384, 8, 1024, 8, "plain"), (6, 6, 16383, 4, 1024, 8, "plain"), (24, 6, 16384, 8, 1024, 8, "plain"),
    (24, 6, 8193, 16, 512, 8, "plain"), (30, 6, 15873, 8, 900, 8, "negative"),
    # 256 threads: more units than two to a compute unit (groups of more than eight heads: than one)
    (17, 17, 300, 8, 19, 8, "plain"), (34, 17, 8192, 8, 300, 8, "plain"), (68, 17, 513, 24, 32, 8, "plain"),
    (180, 9, 700, 8, 44, 8, "plain"), (17, 17, 2048, 8, 1500, 8, "tiny"),
    # groups of more than eight and of more than sixteen heads, one and several workgroups per unit
    (9, 1, 2000, 8, 125, 0, "plain"), (16, 1, 17000, 8, 1062, 0, "plain"), (33, 1, 9000, 8, 562, 0, "plain"),
    (40, 2, 1000, 32, 62, 0, "negative"),
    # more rows in flight: 36 MiB by units for a quarter of the device
    (64, 64, 6144, 32, 384, 0, "plain"),
])
def test_decode_bins_lists_and_variants(Hq, Hkv, L, r, k, cus, scores):
    """The decode launch at the edges of its first-level bins (fine ones around the label query's largest
    value, coarse ones far from it), of its candidate lists and of the rules that choose its form: index
    lists equal to the oracle's, outputs within the parity bounds."""
    t = make_layer_numpy(Workload("t", 1, Hq, Hkv, 128, L, r, k, 1))
    ch = rand_channels(Hkv, r, seed=L + r)
    rng = np.random.default_rng(L + k)
    if scores != "plain":
        for h in range(Hkv):
            x = np.abs(rng.standard_normal((L, r)))
            scale = {"tiny": 1e-6, "huge": 2e4, "negative": -1.0, "front": 1.0}[scores]
            if scores == "front":
                x[L // 5:] -= 4.0
            t["K"][0, h][:, ch[h]] = np.clip(x * scale, -6e4, 6e4).astype(np.float16)
            t["q"].reshape(1, Hkv, Hq // Hkv, 128)[0, h][:, ch[h]] = np.float16(0.01 if scores == "huge" else 0.5)
    if cus:
        ds.ds_pretend_device(cus, 8, 160 << 10)
    try:
        plan = ds.ds_plan_describe(ds.shape(1, Hq, Hkv, 128, L, L, r, k))
        assert plan["scores_itself"] == 1
        if cus:
            assert plan["workgroups_per_unit"] == 1
        full_parity(Case(t["q"], t["K"], t["V"], ch, L, k), what=f"Hq{Hq} Hkv{Hkv} L{L} r{r} k{k} {scores}")
    finally:
        ds.ds_pretend_device(0, 0, 0)


@pytest.mark.parametrize("n,r,inter", [(1, 8, False), (1, 3, True), (15, 24, False), (16, 8, True), (17, 128, False), (40, 12, False)])
def test_append_kv_equals_the_cache_built_in_one_go(n, r, inter):
    """Rows and label values of n new tokens, below, at and above the 16 that a workgroup takes at a time."""
    B, Hkv, L, L_max = 2, 3, 50 + n, 60 + n
    t = make_layer_numpy(Workload("t", B, Hkv, Hkv, 128, L, r, 1, 1), L_max=L_max)
    ch = rand_channels(Hkv, r, seed=n)
    K, V = to_dev(t["K"]), to_dev(t["V"])
    k_new, v_new = K[:, :, 50:L].contiguous(), V[:, :, 50:L].contiguous()
    shp = ds.shape(B, Hkv, Hkv, 128, L, L_max, r, 1)
    label = torch.full((B, Hkv, L_max, r), -7.0, dtype=torch.float16, device="cuda")
    if inter:
        KV = torch.full((B, Hkv, L_max, 2, 128), 5.0, dtype=torch.float16, device="cuda")
        ds.ds_append_kv(k_new, v_new, KV, None, to_dev(ch), label, shp, 50, n, ds.DS_KV_INTERLEAVED)
        Kc, Vc = KV[:, :, :, 0], KV[:, :, :, 1]
    else:
        Kc, Vc = torch.full_like(K, 5.0), torch.full_like(V, 5.0)
        ds.ds_append_kv(k_new, v_new, Kc, Vc, to_dev(ch), label, shp, 50, n, ds.DS_KV_SPLIT)
    torch.cuda.synchronize()
    assert torch.equal(Kc[:, :, 50:L], k_new) and torch.equal(Vc[:, :, 50:L], v_new)
    ref = O.build_label(t["K"], ch, L)
    assert np.array_equal(label[:, :, 50:L].cpu().numpy().view(np.uint16), np.ascontiguousarray(ref[:, :, 50:L]).view(np.uint16))
    for x, v in ((Kc, 5.0), (Vc, 5.0), (label, -7.0)):
        assert (x[:, :, :50] == v).all() and (x[:, :, L:] == v).all()


@pytest.mark.parametrize("cus,Hq,Hkv,L,r", [(2048, 40, 40, 131072, 8), (2048, 120, 40, 131072, 8), (0, 100, 100, 70000, 40)])
def test_workgroups_that_start_late_leave_no_old_output(cus, Hq, Hkv, L, r):
    """More workgroups than the device holds (the planner is told of a larger one) and a poll limit of
    one: the first workgroups of a unit give up and raise its error word, others start only then and leave
    at once.  The unit's output is all NaN then -- no number of an earlier call stays in it -- and every other
    unit's is right."""
    k = L // 16
    w = Workload("t", 1, Hq, Hkv, 128, L, r, k, 1)
    t = make_layer_torch(w, "cuda", layer=0)
    ch = to_dev(rand_channels(Hkv, r, seed=L + r))
    shp = ds.shape(1, Hq, Hkv, 128, L, L, r, k)
    label = torch.empty((1, Hkv, L, r), dtype=torch.float16, device="cuda")
    ds.ds_build_label(t["K"], ch, label, shp)

    def decode(ws):
        out = torch.full((1, Hq, 128), 7.0, dtype=torch.float32, device="cuda")
        ds.ds_sparse_decode(t["q"], label, t["K"], t["V"], ch, out, None, ws, shp)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    good = decode(ds.ds_workspace_alloc(shp))
    try:
        if cus:
            ds.ds_pretend_device(cus, 8, 160 << 10)
        plan = ds.ds_plan_describe(shp)
        assert plan["workgroups"] > (2 if r <= 32 else 4) * 256 and plan["workgroups_per_unit"] > 1 and plan["scores_itself"] == (r <= 32)
        ws = ds.ds_workspace_alloc(shp)
        ds.ds_tune_set(5, 1)
        bad = decode(ws)
        ds.ds_tune_set(5, 0)
        n_failed, _ = ds.ds_workspace_errors(ws, shp)
    finally:
        ds.ds_tune_set(5, 0)
        ds.ds_pretend_device(0, 0, 0)
    failed = np.isnan(bad.reshape(Hkv, -1)).all(axis=1)
    assert int(failed.sum()) == n_failed and (n_failed > 0 or r > 32)
    assert not (bad == 7.0).any()
    ok = np.repeat(~failed, Hq // Hkv)
    if ok.any():
        check_output(bad[0][ok], good[0][ok].astype(np.float64), "units that did not fail")


@pytest.mark.parametrize("ties", [True, False])
@pytest.mark.parametrize("L,n,one", [(4000, 64, ONE), (4000, 65, ONE), (4000, 384, ONE), (4000, 385, ONE), (4000, 512, ONE),
                                     (4000, 513, ONE), (6000, 4097, ONE), (20000, 64, SEVERAL), (20000, 65, SEVERAL),
                                     (20000, 385, SEVERAL), (20000, 1024, SEVERAL), (20000, 1025, SEVERAL)])
def test_decode_settles_any_number_of_candidates(L, n, one, ties):
    """n keys in the threshold bin, equal or not, on both sides of what one lane ranks, one wavefront settles,
    LDS holds and the workgroup reads at a time; the threshold lies in the middle, at the first and at the last of them."""
    rng = np.random.default_rng(L + n)
    t = make_layer_numpy(Workload("t", 1, 1, 1, 128, L, 8, 1, 1))
    ch = rand_channels(1, 8, seed=n)
    # scores 2 (100 tokens), 1 .. 1 + 2^-9 (n tokens), and 1/4
    t["q"][0, 0][ch[0]] = 0.0
    t["q"][0, 0][ch[0][0]], t["q"][0, 0][ch[0][1]] = 1.0, 2.0 ** -9
    lab = np.zeros((L, 8), np.float16)
    lab[:, 0] = 0.25
    where = rng.permutation(L)
    lab[where[:100], 0] = 2.0
    lab[where[100:100 + n], 0] = 1.0
    if not ties:
        lab[where[100:100 + n], 1] = rng.integers(0, 1024, n) / 1024
    t["K"][0, 0][:, ch[0]] = lab
    for k in (101, 100 + n // 2, 100 + n):
        assert (ds.ds_plan_describe(ds.shape(1, 1, 1, 128, L, L, 8, k))["workgroups_per_unit"] == 1) == one or k * 16 > L
        full_parity(Case(t["q"], t["K"], t["V"], ch, L, k), check_dense=False, what=f"{n} candidates of {L}, k {k}")
