"""Grouping by bins (one workgroup per bin of the top key bits): sizes at the edges of its tiles, of its LDS sort and of
the route itself, and the takeover of bins whose own workgroups do not run.  Integer outputs, compared exactly."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2411_08446_amd as lsh
import paper_2411_08446_amd.binding as binding
from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    gpu_harness.lsh.load_library()
    return gpu_harness


# the key is 2 expert bits and L * 5 bucket bits; bin: its top 8 bits
@pytest.mark.parametrize("in_bin", [1, 63, 64, 65, 1023, 1025, 4095, 4096, 4097, 8191, 12289])
@pytest.mark.parametrize("L,distinct", [(3, 5), (3, 4000), (6, 40), (6, 100000)])   # one radix pass; sub-bins or several passes
def test_bin_sizes(H, in_bin, L, distinct):
    # one bin of in_bin keys among 5000 others: around a wave, a round of the workgroup and the LDS sort's limit,
    # with few different keys (crowded sub-bins), and with nearly all different
    d, dtype, E, r = 8, "bf16", 4, 16
    rng = np.random.default_rng(in_bin * 10 + L + distinct)
    low = 5 * L - 6
    N = in_bin + 5000
    ids = rng.integers(0, 1 << (5 * L), N, dtype=np.uint64)
    expert = rng.integers(0, E, N)
    where = rng.permutation(N)[:in_bin]
    expert[where] = 2
    ids[where] = (np.uint64(37) << np.uint64(low)) | (rng.integers(0, distinct, in_bin, dtype=np.uint64) % np.uint64(1 << low))
    tokens = synth.f32_to_storage(rng.standard_normal((N, d)).astype(np.float32), dtype)
    rot = np.zeros((L, r, d), tokens.dtype)
    print("case bin of", in_bin, "L", L, "distinct", distinct, flush=True)
    H.run_and_check(tokens, rot, expert.astype(np.int32).reshape(N, 1), E, dtype, lambda c: c, bucket_override=ids, skip_hash=True)


@pytest.mark.parametrize("N", [4096, 65535, 65536, 65537, 131073, 262144, 262145, 524287])
def test_tile_sizes(H, N):
    # the tile of the first launch doubles at 65536, 131072 and 262144 assignments; 4096 is one bin
    d, dtype, E, L, r = 8, "bf16", 300, 3, 8                        # 9 expert bits: a bin holds several experts
    rng = np.random.default_rng(N)
    pool = rng.integers(0, 16 ** 3, max(1, N // 3), dtype=np.uint64)
    tokens = synth.f32_to_storage(rng.standard_normal((N, d)).astype(np.float32), dtype)
    rot = np.zeros((L, r, d), tokens.dtype)
    expert = np.minimum(rng.integers(0, E, (N, 1)), rng.integers(0, E, (N, 1))).astype(np.int32)
    print("case tiles N", N, flush=True)
    H.run_and_check(tokens, rot, expert, E, dtype, lambda c: c, bucket_override=pool[rng.integers(0, pool.size, N)], skip_hash=True)


@pytest.mark.parametrize("first_bin", [1, 37, 255])
@pytest.mark.parametrize("skew", [False, True])                     # True: one bin of 6000 keys, sorted in global memory
def test_bins_whose_workgroups_do_not_run_are_taken_over(first_bin, skew):
    # The workgroups of the bins below first_bin leave at once; the others find those bins open, claim them one by one
    # and do them before their own.  Every output equals that of the ordinary call.
    lib = lsh.load_library()
    E, L, r, d, N = 4, 4, 16, 8, 20000
    rng = np.random.default_rng(first_bin)
    expert = rng.integers(0, E, (N, 1)).astype(np.int32)
    ids = rng.integers(0, 3000, N).astype(np.int64) * 333
    if skew:
        expert[:6000], ids[:6000] = 0, rng.integers(0, 1000, 6000)
    x = torch.from_numpy(rng.standard_normal((N, d)).astype(np.float32)).cuda()
    et, bt = torch.from_numpy(expert).cuda(), torch.from_numpy(ids).cuda()
    outs = []
    for take_over in (False, True):
        o = lsh.CompressOutputs.allocate(N, d, 1, E, L, r, torch.float32)
        for t in (o.centroids, o.seg_offsets, o.seg_expert, o.expert_offsets, o.perm, o.seg_of, o.num_segments):
            t.fill_(-7)
        o.workspace.fill_(0xA5)
        print("case takeover first_bin", first_bin, "skew", skew, take_over, flush=True)
        if take_over:
            ws, ws_bytes = binding._aligned_ws(o.workspace)
            p = lambda t: ctypes.c_void_p(t.data_ptr())
            status = lib.lshmoe_test_compress_takeover(
                p(x), p(et), p(bt), ctypes.c_int64(N), d, 1, E, L, r, lsh.LSHMOE_F32, p(o.centroids), p(o.seg_offsets),
                p(o.seg_expert), p(o.expert_offsets), p(o.perm), p(o.seg_of), p(o.num_segments), ctypes.c_void_p(ws),
                ctypes.c_size_t(ws_bytes), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                ctypes.c_uint32(first_bin), ctypes.c_uint32(2))
            assert status == lsh.LSHMOE_OK
        else:
            lsh.lshmoe_compress(x, et, bt, E, L, r, o)
        torch.cuda.synchronize()
        outs.append(o)
    a, b = outs
    for name in ("num_segments", "seg_offsets", "seg_expert", "expert_offsets", "perm", "seg_of", "centroids"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


def _skewed(name, rng):
    """Keys of which most share a few bins: (experts [N], ids [N], E, L, r)."""
    E, L, r, N = 4, 6, 16, 40000                        # 2 expert bits, 30 bucket bits: a bin is 6 bucket bits
    ids = rng.integers(0, 1 << 30, N, dtype=np.uint64)
    expert = np.full(N, 2)
    base = np.uint64(37 << 24)
    narrow = base | rng.integers(0, 1 << 24, N, dtype=np.uint64)
    if name == "one bin":
        ids = narrow
    elif name == "one bin, few keys":                   # clusters that steps of the sample fall into
        ids = base | (rng.integers(0, 9, N, dtype=np.uint64) * np.uint64(999))
    elif name == "last bin":
        expert, ids = np.full(N, 3), ids | np.uint64(63 << 24)
    elif name == "first and last key":
        expert = np.where(rng.random(N) < 0.5, 0, 3)
        ids = np.where(expert == 0, np.uint64(0), np.uint64((1 << 30) - 1))
        some = rng.random(N) < 0.3
        ids = np.where(some & (expert == 0), ids + rng.integers(0, 1 << 20, N, dtype=np.uint64), ids)
        ids = np.where(some & (expert == 3), ids - rng.integers(0, 1 << 20, N, dtype=np.uint64), ids)
    elif name == "two frequent keys":
        u = rng.random(N)
        ids = np.where(u < 0.4, base | np.uint64(5), np.where(u < 0.7, base | np.uint64(1 << 23), narrow))
    elif name == "a frequent key among many":           # below the share that makes the bin one workgroup's
        ids = np.where(rng.random(N) < 0.6, base | np.uint64(1 << 22), narrow)
    elif name == "several experts per bin":             # 9 expert bits: two experts share a bin
        E = 300
        expert = np.where(rng.random(N) < 0.8, rng.integers(100, 104, N), rng.integers(0, E, N))
        ids = rng.integers(0, 1 << 30, N, dtype=np.uint64)
    elif name == "every bin large":
        N = 524288
        expert, ids = rng.integers(0, 4, N), rng.integers(0, 1 << 30, N, dtype=np.uint64) & np.uint64(0x30ffffff)
    elif name == "the sample misses":                   # every 16th key of the bin is spread out, the rest is narrow
        N = 16384
        expert = np.full(N, 2)
        ids = base | np.uint64(1 << 22) | rng.permutation(N).astype(np.uint64)
        ids[8::16] = base | (np.arange(N // 16, dtype=np.uint64) * np.uint64(16000))
    elif name == "the sample misses, frequent":         # ... and mostly two keys, none of them at a step
        N = 16384
        expert = np.full(N, 2)
        ids = base | np.uint64(1 << 22) | np.where(rng.random(N) < 0.5, np.uint64(77), np.uint64(99))
        ids[8::16] = base | (np.arange(N // 16, dtype=np.uint64) * np.uint64(16000))
    elif name == "the sample shows one key":            # ... that is one in sixteen of the bin
        N = 16384
        expert = np.full(N, 2)
        ids = base | np.uint64(1 << 22) | rng.permutation(N).astype(np.uint64)
        ids[8::16] = base | np.uint64(5 << 20)
    elif name == "eight key bits":
        E, L, r = 2, 1, 64                              # the bin is the key
        expert, ids = np.where(rng.random(N) < 0.7, 1, 0), np.where(rng.random(N) < 0.5, 127, rng.integers(0, 128, N)).astype(np.uint64)
    return expert, ids.astype(np.uint64), E, L, r


@pytest.mark.parametrize("name", ["one bin", "one bin, few keys", "last bin", "first and last key", "two frequent keys",
                                  "a frequent key among many", "several experts per bin", "every bin large",
                                  "the sample misses", "the sample misses, frequent", "the sample shows one key",
                                  "eight key bits"])
def test_large_bins_in_parts(H, name):
    rng = np.random.default_rng(len(name))
    expert, ids, E, L, r = _skewed(name, rng)
    d, dtype, N = 8, "bf16", expert.size
    tokens = synth.f32_to_storage(rng.standard_normal((N, d)).astype(np.float32), dtype)
    print("case large bins:", name, flush=True)
    H.run_and_check(tokens, np.zeros((L, r, d), tokens.dtype), expert.astype(np.int32).reshape(N, 1), E, dtype, lambda c: c,
                    bucket_override=ids, skip_hash=True)


def _compare_with_takeover(expert, ids, E, L, r, first_bin):
    """Every output of a call whose first workgroups leave at once equals that of the ordinary call."""
    lib = lsh.load_library()
    N, d = expert.size, 8
    x = torch.randn(N, d, device="cuda")
    et = torch.from_numpy(expert.astype(np.int32).reshape(N, 1)).cuda()
    bt = torch.from_numpy(ids.view(np.int64)).cuda()
    a, b = (lsh.CompressOutputs.allocate(N, d, 1, E, L, r, torch.float32) for _ in range(2))
    names = ("num_segments", "seg_offsets", "seg_expert", "expert_offsets", "perm", "seg_of", "centroids")
    for o in (a, b):
        for n in names:
            getattr(o, n).fill_(-7)
        o.workspace.fill_(0xA5)
    lsh.lshmoe_compress(x, et, bt, E, L, r, a)
    ws, ws_bytes = binding._aligned_ws(b.workspace)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    status = lib.lshmoe_test_compress_takeover(
        p(x), p(et), p(bt), ctypes.c_int64(N), d, 1, E, L, r, lsh.LSHMOE_F32, p(b.centroids), p(b.seg_offsets),
        p(b.seg_expert), p(b.expert_offsets), p(b.perm), p(b.seg_of), p(b.num_segments), ctypes.c_void_p(ws),
        ctypes.c_size_t(ws_bytes), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
        ctypes.c_uint32(first_bin), ctypes.c_uint32(2))
    assert status == lsh.LSHMOE_OK
    torch.cuda.synchronize()
    for n in names:
        assert torch.equal(getattr(a, n), getattr(b, n)), n


@pytest.mark.parametrize("first_bin", [1, 37, 200])
@pytest.mark.parametrize("name", ["one bin", "two frequent keys", "the sample misses"])
def test_parts_whose_workgroups_do_not_run_are_taken_over(name, first_bin):
    # bin 165 is large, its parts belong to the workgroups of the first bins: those that run claim them while they wait
    rng = np.random.default_rng(first_bin)
    expert, ids, E, L, r = _skewed(name, rng)
    expert[-500:] = 3                                   # work behind the large bin, too
    print("case parts taken over:", name, first_bin, flush=True)
    _compare_with_takeover(expert, ids, E, L, r, first_bin)


def test_large_bins_of_changing_sizes(H):
    # The same result every time, whatever the call before has left in LDS: large bins of several sizes (more than 65536
    # keys draw a larger sample) and a balanced input in turn.  The workgroups of a bin's parts must agree on the parts'
    # ranges to the key.
    rng = np.random.default_rng(17)
    E, L, r = 4, 6, 16                                  # 2 expert bits, 30 bucket bits: a bin is 6 bucket bits
    cases = []
    for N, spread in ((131072, 1 << 24), (20000, 1 << 24), (80000, 1 << 24), (16384, 1 << 30)):
        ids = rng.integers(0, spread, N, dtype=np.uint64)
        expert = np.full(N, 2) if spread == 1 << 24 else rng.integers(0, E, N)
        x = torch.randn(N, 8, device="cuda")
        et = torch.from_numpy(expert.astype(np.int32).reshape(N, 1)).cuda()
        bt = torch.from_numpy(ids.view(np.int64)).cuda()
        cases.append((x, et, bt, lsh.CompressOutputs.allocate(N, 8, 1, E, L, r, torch.float32), []))
    for call in range(30):
        for x, et, bt, o, first in cases:
            lsh.lshmoe_compress(x, et, bt, E, L, r, o)
            S = int(o.num_segments)
            got = [o.num_segments.clone(), o.perm.clone(), o.seg_of.clone(), o.seg_offsets[:S + 1].clone(),
                   o.seg_expert[:S].clone(), o.expert_offsets.clone(), o.centroids[:S].clone()]
            if not first:
                key = (et[:, 0].long() << 40) + bt
                assert S == int(torch.unique(key).numel())
                first.extend(got)
            for a, b in zip(got, first):
                assert torch.equal(a, b), "call %d of %d assignments" % (call, x.shape[0])
