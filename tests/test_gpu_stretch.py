"""Rows dealt by columns (restore, restore + combine, token gradient on large clusters) against the same calls on parts of the tokens
that are too few for it: a token's row depends on nothing else, so the results agree bit for bit.  The parts run the way
that the other tests hold to the oracle."""
import pytest
import torch

import paper_2411_08446_amd as lsh

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _clusters(T, k, share, gen):
    """Random clusters of N = T k assignments, every one with members: seg_of and seg_offsets, whose rest is garbage."""
    N = T * k
    if isinstance(share, tuple):                         # so many alone, the rest in six large clusters that come last
        alone = int(N * share[0])
        seg = torch.cat([torch.arange(alone, device="cuda"), alone + torch.randint(6, (N - alone,), device="cuda", generator=gen)])
        seg = seg[torch.randperm(N, device="cuda", generator=gen)]
    else:
        seg = torch.randint(max(1, int(N * share)), (N,), device="cuda", generator=gen)
    _, seg = torch.unique(seg, return_inverse=True)
    size = torch.bincount(seg)
    off = torch.full((N + 1,), 0x7f7f7f7f, dtype=torch.int32, device="cuda")
    off[0] = 0
    off[1:size.numel() + 1] = torch.cumsum(size, 0)
    return seg.to(torch.int32), off, size


def _rows(n, d, dt, gen):
    return torch.randn(n, d, device="cuda", generator=gen).to(dt)


# rows of four, eight, twelve and sixteen stretches; tokens off the grid of a workgroup, of a part and of a lane group.  Which
# of them go by columns: tests/host_sanitize/stretch_plan.cpp
SHAPES = [("bf16", 512, 8192 + 13, 1), ("bf16", 1024, 4096, 2), ("bf16", 1024, 8192 + 1, 3), ("bf16", 1536, 4096 + 31, 2),
          ("bf16", 2048, 4096 + 33, 4), ("f32", 256, 8192 + 7, 2), ("f32", 1024, 4096 + 65, 1), ("bf16", 1024, 4096 + 5, 5),
          ("bf16", 768, 8192 + 3, 2), ("bf16", 512, 16384 + 13, 1), ("f32", 1024, 4096 + 65, 2)]


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("dtype,d,T,k", SHAPES)
def test_combine_by_columns(dtype, d, T, k, flags):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d + k)
    dt = DTYPES[dtype]
    for share, with_offsets in ((0.002, True), (0.1, True), (0.1, False), (0.9, True), (0.14, True), (0.14, False), (0.2, True),
                                ((0.14,), True), ((0.14,), False)):
        print("case combine", dtype, d, T, k, flags, share, with_offsets, flush=True)
        seg, off, size = _clusters(T, k, share, gen)
        S = size.numel()
        x, c, e = _rows(T, d, dt, gen), _rows(S, d, dt, gen), _rows(S, d, dt, gen)
        w = torch.rand(T, k, device="cuda", generator=gen)
        got, want = torch.zeros(T, d, dtype=dt, device="cuda"), torch.ones(T, d, dtype=dt, device="cuda")
        lsh.lshmoe_decompress_combine(x, c, e, seg, off if with_offsets else None, w, got, flags)
        for a in range(0, T, 1000):                      # at most 8 MB of rows: not dealt by columns
            b = min(a + 1000, T)
            lsh.lshmoe_decompress_combine(x[a:b], c, e, seg[a * k:b * k], off if with_offsets else None, w[a:b], want[a:b], flags)
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
        # a few tokens in binary64, so that both are not wrong alike
        t = torch.randint(T, (32,), device="cuda", generator=gen)
        s = seg.view(T, k)[t].long()
        y = e[s].double()
        if flags == 0:
            res = x[t].double()[:, None] - c[s].double()
            y = y + (torch.where((size[s] == 1)[..., None], 0.0, res) if with_offsets else res)
        ref = (w[t].double()[..., None] * y).sum(1)
        tol = 2.0 ** -7 if dtype == "bf16" else 1e-5    # one unit of the last place of bf16; binary32 sums of k terms
        assert float((got[t].double() - ref).abs().max()) <= tol * float(ref.abs().max())


GRAD_SHAPES = [("bf16", 512, 32768 + 13, 2), ("bf16", 1024, 32768 + 1, 1), ("bf16", 1024, 16384 + 31, 2), ("bf16", 1536, 8192 + 7, 3),
               ("f32", 1024, 16384 + 33, 2), ("bf16", 2048, 4096 + 5, 4), ("bf16", 1024, 8192 + 3, 5), ("f32", 1024, 32768 + 3, 1),
               ("f32", 512, 32768 + 33, 2)]


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("dtype,d,T,k", GRAD_SHAPES)
def test_token_gradient_by_columns(dtype, d, T, k, flags):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d + k)
    dt = DTYPES[dtype]
    for share in (0.002, 0.12, 0.9, (0.14,)):
        print("case gradient", dtype, d, T, k, flags, share, flush=True)
        seg, off, size = _clusters(T, k, share, gen)
        S = size.numel()
        g, h, gs = _rows(T * k, d, dt, gen), _rows(S, d, dt, gen), _rows(S, d, dt, gen)
        got, want = torch.zeros(T, d, dtype=dt, device="cuda"), torch.ones(T, d, dtype=dt, device="cuda")
        lsh.lshmoe_compress_backward(None if flags else g, h, None if flags else gs, seg, off, k, got, flags)
        for a in range(0, T, 1000):
            b = min(a + 1000, T)
            lsh.lshmoe_compress_backward(None if flags else g[a * k:b * k], h, None if flags else gs, seg[a * k:b * k], off, k,
                                         want[a:b], flags)
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
        t = torch.randint(T, (32,), device="cuda", generator=gen)
        s = seg.view(T, k)[t].long()
        n = size[s].double()[..., None]
        if flags:
            y = h[s].double() / n
        else:
            y = torch.where(n == 1, h[s].double(), g.view(T, k, d)[t].double() + (h[s].double() - gs[s].double()) / n)
        ref = y.sum(1)
        tol = 2.0 ** -7 if dtype == "bf16" else 1e-5
        assert float((got[t].double() - ref).abs().max()) <= tol * float(ref.abs().max())


# 24 to 256 MB of output in rows of 2 KB and two to four experts go by columns at the smaller shares, the others do not
@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("dtype,d,T,k", [("bf16", 1024, 16384, 2), ("bf16", 1024, 32768, 2), ("bf16", 1024, 16384 + 13, 3),
                                         ("f32", 512, 8192 + 1, 4), ("bf16", 1024, 16383, 2), ("bf16", 1024, 32769, 2),
                                         ("bf16", 512, 12288 + 5, 2), ("bf16", 1024, 6144 + 5, 2), ("bf16", 1024, 6144 - 1, 2),
                                         ("bf16", 1536, 8192 + 3, 2),
                                         ("bf16", 1024, 65536 + 1, 2)])
def test_restore_by_columns(dtype, d, T, k, flags):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d + k)
    dt = DTYPES[dtype]
    for share, with_offsets in ((0.002, True), (0.1, True), (0.1, False), (0.3, True), (0.06, True), ((0.06,), True), ((0.06,), False)):
        print("case restore", dtype, d, T, k, flags, share, with_offsets, flush=True)
        seg, off, size = _clusters(T, k, share, gen)
        S = size.numel()
        perm = torch.sort(seg, stable=True)[1].to(torch.int32)
        count = torch.tensor([S], dtype=torch.int32, device="cuda")
        x, c, e = _rows(T, d, dt, gen), _rows(S, d, dt, gen), _rows(S, d, dt, gen)
        got, want = torch.zeros(T, k, d, dtype=dt, device="cuda"), torch.ones(T, k, d, dtype=dt, device="cuda")
        given = off if with_offsets else None
        lsh.lshmoe_decompress(x, c, e, seg, given, k, got, flags, perm=perm, num_segments=count)
        lsh.lshmoe_decompress(x, c, e, seg, given, k, want, flags)      # without the count: assignment order, row by row
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
        t = torch.randint(T, (32,), device="cuda", generator=gen)
        s = seg.view(T, k)[t].long()
        y = e[s].double()
        if flags == 0:
            res = x[t].double()[:, None] - c[s].double()
            y = y + (torch.where((size[s] == 1)[..., None], 0.0, res) if with_offsets else res)
        tol = 2.0 ** -7 if dtype == "bf16" else 1e-6    # one unit of the last place of bf16; two binary32 roundings
        assert float((got[t].double() - y).abs().max()) <= tol * float(y.abs().max())
