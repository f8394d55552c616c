"""Every workgroup tile of the tiled kernel against 64-bit torch, on calls that the dispatch gives it."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def agq():
    from paper_2312_05693_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def tile_of(agq):
    """tile_of(M, K, Ns, n_extra): 100 x 16-token tiles + 10 x (channels / 64) + groups, + 1000 x the slices of a K split; -1: the
    weight-streaming kernel."""
    from paper_2312_05693_amd import build
    probe = ctypes.CDLL(build.PROBE_LIB)

    def tile(M, K, Ns, n_extra=-1, workspace_bytes=0, x_kind=1):
        return probe.agq_probe_gemm_tile(x_kind, ctypes.c_int64(M), ctypes.c_int64(K), (ctypes.c_int64 * len(Ns))(*Ns), len(Ns), n_extra,
                                         ctypes.c_size_t(workspace_bytes))
    return tile


def inputs(M, K, N, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q = torch.randint(-128, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    wq = torch.randint(-8, 8, (N, K), generator=g, device="cuda", dtype=torch.int8)
    sw = torch.rand(N, generator=g, device="cuda").half() * 0.01 + 0.001
    return g, q, wq, sw


def check(acc, y, q64, wq, sw, e):
    want = torch.mm(q64, wq.double().t().contiguous())                   # whole numbers below 2^53: exact
    assert torch.equal(acc.double(), want)
    ref = want * (sw.double() * 2.0 ** e)
    # one rounding to fp16 (2^-11, or half of the smallest subnormal), of an fp32 product of two factors that are rounded to fp32 (3 x 2^-24)
    assert bool(((y.double() - ref).abs() <= ref.abs() * (2.0 ** -11 + 2.0 ** -22) + 2.0 ** -25).all())


# token counts one past and at the edge of a tile, widths that end inside a wavefront's channels and off the 16-byte grid, and
# K steps around the number that a wavefront requests ahead (P of the kernel): fewer, as many, one more, a remainder of each size
CASES = [
    (211, 17, 44, (1, 2, 9, 10, 11)), (211, 64, 513, (3, 8)), (221, 32, 22000, (1, 5, 7)), (221, 129, 12001, (12, 14, 20)),
    (411, 33, 8200, (2, 6, 7, 8, 11)), (421, 33, 22001, (6, 7, 8, 11)), (431, 65, 22000, (1, 4, 5, 6, 7, 11, 13)),
    (441, 257, 12000, (1, 3, 4, 5, 6, 9, 14)), (821, 257, 10000, (1, 5, 6, 7, 8)), (821, 1100, 2001, (9, 12, 13, 14)),
    (831, 161, 22000, (3, 4, 5, 6)), (831, 1100, 10000, (1,)), (841, 513, 12000, (1, 2, 3, 4, 5, 6, 7, 9)),
    (212, 17, 44, (12, 15, 16, 17, 18, 19)), (222, 17, 22000, (12, 13, 14, 15)), (412, 33, 8201, (12, 13, 18, 20)),
    (422, 33, 22000, (12, 13, 20)), (422, 400, 4096, (19,)), (4411, 17, 40, (20, 21, 26)), (4421, 1100, 300, (64, 66, 67)),
    (3421, 1050, 512, (64,)),
    # a last round of 128 x 256 tiles that is dealt out as halves (some of them past the last channel)
    (841, 1100, 17000, (2, 5, 8)), (841, 2000, 10003, (3,)),
    # token tiles that start apart in K: the first and the last of a group's steps, odd and even counts of them, a short second group
    (212, 100, 4096, (85, 86)), (222, 213, 4096, (85, 86)), (422, 300, 4096, (24, 85, 86)), (422, 100, 8201, (41, 42)),
]


@pytest.mark.parametrize("tile,M,N,steps", [(t, M, N, s) for t, M, N, every in CASES for s in every])
def test_tile(agq, tile_of, tile, M, N, steps):
    K = 128 * steps
    size = agq.gemm_workspace_bytes(M, N, K)
    assert tile_of(M, K, [N], workspace_bytes=size) == tile
    _, q, wq, sw = inputs(M, K, N, 7 * steps + M)
    acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
    ybuf = torch.full((M, N + 3), 5.0, dtype=torch.float16, device="cuda")           # a pitch off the 16-byte grid
    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    agq.gemm_w4a8(q, -4, agq.pack_w4(wq), sw, N, K, x_kind=agq.AGQ_X_Q, acc_out=acc, y=ybuf[:, :N], workspace=ws)
    check(acc, ybuf[:, :N], q.double(), wq, sw, -4)
    assert bool((ybuf[:, N:] == 5.0).all())


@pytest.mark.parametrize("tile,M,N,steps,n_extra", [(841, 513, 12000, 8, 3), (841, 1100, 17000, 4, 2), (841, 513, 12000, 1, 1), (831, 161, 22000, 5, 2),
                                                    (821, 1100, 2001, 11, 2), (441, 257, 12000, 9, 4), (431, 65, 22000, 6, 2),
                                                    (421, 33, 22000, 5, 5), (221, 32, 22000, 3, 6), (412, 33, 8200, 9, 4),
                                                    (212, 17, 44, 14, 3), (222, 17, 22000, 13, 4), (422, 300, 4096, 14, 3)])
def test_tile_with_extra_steps(agq, tile_of, tile, M, N, steps, n_extra):
    """TRIP blobs: the shifts behind the extra steps, which may be all of the steady loop, and its tail."""
    K = 128 * steps
    g, _, wq, sw = inputs(M, K, N, 11 * steps + M)
    x = torch.randn(M, K, generator=g, device="cuda").half()
    levels = [4, 3, 2, 1]
    alpha = torch.zeros(K, dtype=torch.int8)
    order = torch.Generator()
    order.manual_seed(13 * steps + M)
    left = list(torch.randperm(K, generator=order).tolist())
    for c in range(n_extra):                                             # one chunk more for every channel past a multiple of 128
        for k in left[:1 if c < 4 else 128]:
            alpha[k] = levels[c % 4] if c < 4 else levels[(c - 4) % 4]
        left = left[1 if c < 4 else 128:]
    packed, extra = agq.pack_w4_trip(wq, alpha.numpy())
    assert extra == n_extra
    size = agq.lib().agq_gemm_trip_workspace_bytes(M, N, K, extra)
    assert tile_of(M, K, [N], extra, size) == tile
    e = -6
    acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
    y = torch.empty(M, N, dtype=torch.float16, device="cuda")
    agq.gemm_trip_multi(x, 8, e, [(packed, sw, N, y, acc)], extra, K, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    up = 2.0 ** alpha.to("cuda").double()
    q64 = (x.double() * 2.0 ** -e / up).round().clamp(-128, 127) * up
    check(acc, y, q64, wq, sw, e)


@pytest.mark.parametrize("tile,M,Ns,steps,bits,zp,n_extra", [
    # the last round of 128 x 256 tiles, dealt out as halves: its first tile is another projection's than the last whole one, or
    # lies inside a projection, and the projections behind it start among the halves
    (841, 1000, [8101, 8104, 3001, 130], 4, 8, 131, None), (841, 1023, [16300, 4001], 5, 4, 9, None), (841, 1000, [13801, 13825], 2, 8, 7, None),
    (841, 1000, [16301, 3000, 520], 3, 8, 0, 3), (841, 1020, [8100, 8101, 4001], 2, 4, 5, 2),
    # the unsigned grid on the tiles of 32 tokens, and on two groups
    (211, 17, [44, 301], 3, 8, 77, None), (221, 213, [4096, 300], 5, 4, 15, None), (212, 17, [513, 130], 14, 8, 200, None),
    (222, 213, [4096, 300], 20, 4, 1, None), (422, 300, [4096, 300], 14, 8, 128, None), (412, 100, [4096, 300], 14, 8, 3, 3)])
def test_tile_of_several_projections(agq, tile_of, tile, M, Ns, steps, bits, zp, n_extra):
    K = 128 * steps
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * steps + M)
    x = (torch.randn(M, K, generator=g, device="cuda") * 3).half()
    e = -6 if bits == 8 else -1
    alpha = torch.zeros(K, dtype=torch.int8)
    for c in range(n_extra or 0):                                        # as many chunks, of factors 2 and 1 or 3, 2 and 1
        alpha[5 * c + 1::97] = n_extra - c
    projs, weights = [], []
    for i, N in enumerate(Ns):
        _, _, wq, sw = inputs(16, K, N, N + steps + i)
        blob = agq.pack_w4(wq) if n_extra is None else agq.pack_w4_trip(wq, alpha.numpy())
        if n_extra is not None:
            assert blob[1] == n_extra
            blob = blob[0]
        projs.append((blob, sw, N, torch.empty(M, N, dtype=torch.float16, device="cuda"), torch.full((M, N), -7, dtype=torch.int32, device="cuda")))
        weights.append(wq)
    if n_extra is None:
        xq = agq.quantize_act(x, bits, e, zp)
        size = agq.gemm_workspace_bytes(M, sum(Ns), K)
        assert tile_of(M, K, Ns, workspace_bytes=size) == tile
        multi = agq.gemm_w4a8_multi if bits == 8 else agq.gemm_w4a4_multi
        multi(xq, e, projs, K, x_kind=agq.AGQ_X_Q, workspace=torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda"), zp=zp)
    else:
        size = agq.lib().agq_gemm_trip_workspace_bytes(M, sum(Ns), K, n_extra)
        assert tile_of(M, K, Ns, n_extra, size) == tile
        agq.gemm_trip_multi(x, bits, e, projs, n_extra, K, workspace=torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda"), zp=zp)
    lo, hi = (0, 2 ** bits - 1) if zp else (-2 ** (bits - 1), 2 ** (bits - 1) - 1)
    up = 2.0 ** alpha.to("cuda").double()
    q64 = (((x.double() * 2.0 ** -e / up).round() + zp).clamp(lo, hi) - zp) * up
    for (_, sw, _, y, acc), wq in zip(projs, weights):
        check(acc, y, q64, wq, sw, e)


@pytest.mark.parametrize("K,slices", [(4096, 3), (6144, 4)])
def test_split_whose_first_slice_is_the_extra_steps(agq, tile_of, K, slices):
    """Sixteen extra steps, the first slice of the K split to the step: its last step is followed by a shift, and no step of the
    main weights is."""
    M, N, n_extra = 100, 300, 16
    size = agq.lib().agq_gemm_trip_workspace_bytes(M, N, K, n_extra)
    tile = tile_of(M, K, [N], n_extra, size, x_kind=0)
    assert tile // 1000 == slices and -(-(K // 128 + n_extra) // slices) == n_extra          # steps a slice, as the choice divides them
    g, _, wq, sw = inputs(16, K, N, K)
    x = torch.randn(M, K, generator=g, device="cuda").half()
    for counts in ((2048, 0, 0, 0), (700, 600, 300, 256)):               # channels of factor 4, 3, 2, 1: one level, four of them
        alpha = torch.zeros(K, dtype=torch.int8)
        order = torch.Generator()
        order.manual_seed(K)
        left = torch.randperm(K, generator=order)
        for level, n in zip((4, 3, 2, 1), counts):
            alpha[left[:n]] = level
            left = left[n:]
        packed, extra = agq.pack_w4_trip(wq, alpha.numpy())
        assert extra == n_extra
        acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
        y = torch.empty(M, N, dtype=torch.float16, device="cuda")
        agq.gemm_trip_multi(x, 8, -7, [(packed, sw, N, y, acc)], extra, K, workspace=torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda"))
        up = 2.0 ** alpha.to("cuda").double()
        check(acc, y, (x.double() * 2.0 ** 7 / up).round().clamp(-128, 127) * up, wq, sw, -7)


@pytest.mark.parametrize("M,steps,Ns,bits,zp", [(30, 87, [3040], 8, 0), (39, 65, [40, 1264], 8, 0), (255, 85, [400], 8, 131), (17, 74, [801], 4, 0),
                                                (130, 108, [17, 48], 4, 9), (49, 52, [1000], 8, 0)])
def test_row_groups_on_a_long_k(agq, tile_of, M, steps, Ns, bits, zp):
    """Sixteen rows a workgroup over more K steps than its wavefronts hold at a time, ragged last groups and widths."""
    K = 128 * steps
    assert tile_of(M, K, Ns, workspace_bytes=agq.gemm_workspace_bytes(M, sum(Ns), K), x_kind=0) == -1
    g = torch.Generator(device="cuda")
    g.manual_seed(steps + M)
    x = (torch.randn(M, K, generator=g, device="cuda") * 3).half()
    e = -4 if bits == 8 else 0
    projs, weights = [], []
    for N in Ns:
        _, _, wq, sw = inputs(16, K, N, N + steps)
        projs.append((agq.pack_w4(wq), sw, N, torch.empty(M, N, dtype=torch.float16, device="cuda"), torch.full((M, N), -7, dtype=torch.int32, device="cuda")))
        weights.append(wq)
    (agq.gemm_w4a8_multi if bits == 8 else agq.gemm_w4a4_multi)(x, e, projs, K, zp=zp)
    lo, hi = (0, 2 ** bits - 1) if zp else (-2 ** (bits - 1), 2 ** (bits - 1) - 1)
    q64 = ((x.double() * 2.0 ** -e).round() + zp).clamp(lo, hi) - zp
    for (_, sw, _, y, acc), wq in zip(projs, weights):
        check(acc, y, q64, wq, sw, e)
