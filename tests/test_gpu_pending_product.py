"""Products left in the workspace as a sum of planes (ssnet_*_product_*) and the calls that consume
them with d_c = NULL: every output, opened value and message against the oracle's chain
convolution / dense layer -> degree reduction -> truncation (-> ReLU, -> REC), bit for bit.
Shapes cover one whole tile per workgroup, contractions split over several workgroups (several
planes), ragged edges, operands of at most 16 rows, and tensors on both sides of the size limits at
which the reduction changes kernels."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2406_02629_amd import SSNet, SSNetError, binding
from util import field_uniform, to_dev, to_np

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def small_secrets(shape, seed, bits, p):
    """signed values below 2^bits as field elements"""
    v = np.random.default_rng(seed).integers(-(1 << bits), 1 << bits, size=shape, dtype=np.int64)
    return np.where(v < 0, v + p, v).astype(np.uint64)


def check_consumers(s, p, y, shape, leave_product, f=12, seed=0):
    """y: the oracle's product shares [n, B, C, H, W] (degree 2t); leave_product() makes the library's
    product pending.  Runs the consuming calls one after the other, each on a fresh pending product."""
    n, t = s.n, s.t
    k, nr = t + 1, 2 * t + 1
    B, C, H, W = shape
    count = B * C * H * W
    yf = y.reshape(n, count)
    ids = list(range(1, k + 1))
    yr, m1, m2, _ = orc.degree_reduce(yf, n, t, p, seed, 3, full=True)
    yt, u, wsh = orc.truncate(yr, n, t, f, p, seed, 3, full=True)
    rec = orc.reconstruct(yt, ids, p)
    o = np.cumsum([0, nr * k, k * n, k, n]) * count

    # reduction alone, with its two message arrays
    leave_product()
    out = torch.empty((n, count), dtype=torch.int64, device="cuda")
    s.degree_reduce(None, stream_id=3, out=out)
    ws = to_np(s.messages()[: o[2]])
    assert np.array_equal(to_np(out), yr)
    assert np.array_equal(ws[: o[1]].reshape(nr, k, count), m1) and np.array_equal(ws[o[1]:].reshape(k, n, count), m2)

    # reduction + truncation + opening in one launch, all four message arrays
    leave_product()
    out2, got_rec = s.degree_reduce_truncate_reconstruct(None, stream_id=3, ids=ids, out=out)
    ws = to_np(s.messages()[: o[4]])
    for got, ref in zip([ws[o[i]:o[i + 1]] for i in range(4)], (m1, m2, u, wsh)):
        assert np.array_equal(got, ref.reshape(-1))
    assert np.array_equal(to_np(out2), yt) and np.array_equal(to_np(got_rec).reshape(-1), rec)

    # the same pending product again (it stays until the next product call), truncation with the rounding division
    yd = orc.truncate_div(yr, n, t, f, 4, p, seed, 3)
    s.degree_reduce_truncate_div(None, 4, stream_id=3, out=out)
    assert np.array_equal(to_np(out), yd)

    # the shortcut without messages: same residues as the protocol
    leave_product()
    out3, rec3 = s.reduce_truncate_direct(None, stream_id=3, ids=ids, out=out)
    assert np.array_equal(to_np(out3), yt) and np.array_equal(to_np(rec3).reshape(-1), rec)

    # Linear - Truncation - NonLinear tail in one call
    sb, sbi = s.nonlinear_masks((B, C, H, W), stream_id=21)
    osb, osbi = orc.nonlinear_masks(count, n, t, 28, p, seed, 21)
    want = orc.relu(yt, osb, osbi, n, t, p)
    leave_product()
    out5 = torch.empty((n, B, C, H, W), dtype=torch.int64, device="cuda")
    _, planes = s.reduce_truncate_relu(None, 3, sb, sbi, out=out5, want_planes=(C % 64 == 0))
    assert np.array_equal(to_np(out5).reshape(n, -1), want)
    if planes is not None:
        per = planes.numel() // n
        data = (8 if p == binding.P61 else 6) * count + 16
        ref = s.split_planes(to_dev(want.reshape(n, B, C, H, W)))
        assert bool(torch.equal(planes.view(n, per)[:, :data], ref.view(n, per)[:, :data]))

    # the same tail in one pass without messages: the protocol's residues, shares and planes
    leave_product()
    out6 = torch.empty_like(out5)
    _, planes6 = s.reduce_truncate_relu_direct(None, sb, sbi, out=out6, want_planes=(C % 64 == 0))
    assert np.array_equal(to_np(out6).reshape(n, -1), want)
    if planes6 is not None:
        assert bool(torch.equal(planes6.view(n, per)[:, :data], ref.view(n, per)[:, :data]))


# (tests/test_gemm_plan.py holds the kernel and the planes that each of the products here is computed with)
CONV_CASES = [
    # B, C, H, W, Co, k, stride, pad; over the 61-bit prime, five parties:
    (1, 256, 14, 14, 256, 3, 1, 1),     # tiles of 32 x 32, 36 k blocks in four runs, a plane each (seven parties: tiles of 64 x 64, four planes)
    (1, 64, 14, 14, 1024, 1, 1, 0),     # tiles of 32 x 32, more than workgroups at a time, one k block
    (1, 256, 14, 14, 64, 1, 1, 0),      # tiles of 16 x 16, two waves each
    (1, 512, 7, 7, 128, 3, 1, 1),       # 49 pixels: one ragged column tile of 32 x 32, six runs (three and seven parties: eight)
    (2, 128, 9, 7, 65, 3, 2, 1),        # tiles of 32 x 32, ragged rows and columns, stride 2, six runs
    (1, 64, 5, 5, 7, 3, 1, 1),          # at most 16 output channels
    (2, 512, 9, 9, 65, 3, 1, 1),        # over the 45-bit prime too in parts: five runs
]
# tiles of 64 x 64, every one split over several workgroups: up to 16 planes, one pixel to a few columns of tiles
CUT_TILES = {(5, 2, binding.P61): [(1, 1024, 1, 1, 401, 3, 1, 1), (1, 256, 71, 6, 103, 3, 1, 1)], (3, 1, binding.P61): [(1, 1024, 6, 6, 456, 3, 1, 1)],
             (7, 3, binding.P61): [(2, 192, 17, 3, 299, 3, 1, 1)], (5, 2, binding.P45): [(1, 1024, 6, 6, 324, 3, 1, 1)]}


@pytest.mark.parametrize("n,t,p", [(5, 2, binding.P61), (3, 1, binding.P61), (7, 3, binding.P61), (5, 2, binding.P45)])
def test_conv_product_on_planes_then_every_consumer(n, t, p):
    s = SSNet(n, t, f=12, seed=91, p=p)
    bits = 11 if p == binding.P45 else 15
    cases = CONV_CASES[:6] if (n, t, p) == (5, 2, binding.P61) else CONV_CASES[:1] + CONV_CASES[3:5]
    if p == binding.P45:
        cases = cases + CONV_CASES[6:]
    cases = cases + CUT_TILES[n, t, p]
    for (B, C, H, W, Co, k, stride, pad) in cases:
        say("conv product", n, t, hex(p), B, C, H, W, Co, k, stride, pad)
        xs = orc.share(small_secrets((B, C, H, W), 1, bits, p), n, t, p, 91, 5)
        ws = orc.share(small_secrets((Co, C, k, k), 2, bits - 2, p), n, t, p, 91, 6)
        y = orc.conv(xs, ws, stride, pad, p)
        Ho, Wo = y.shape[-2:]
        planes = s.split_planes(to_dev(xs))
        wp = s.pack_weights_conv_taps(to_dev(ws))
        check_consumers(s, p, y, (B, Co, Ho, Wo),
                        lambda: s.conv_product_planes(planes, wp, B, C, H, W, Co, k, k, stride, pad), seed=91)


@pytest.mark.parametrize("n,t,p", [(5, 2, binding.P61), (3, 1, binding.P45)])
def test_prepacked_products_then_every_consumer(n, t, p):
    s = SSNet(n, t, f=12, seed=92, p=p)
    bits = 11 if p == binding.P45 else 15
    for (B, C, H, W, Co) in [(1, 1024, 14, 14, 256), (1, 70, 9, 9, 33), (2, 512, 7, 7, 2048)]:
        say("1x1 product", n, t, hex(p), B, C, H, W, Co)
        x = small_secrets((B, C, H, W), 3, bits, p)
        xs_o = orc.share(x, n, t, p, 92, 6)
        ws = orc.share(small_secrets((Co, C, 1, 1), 4, bits - 2, p), n, t, p, 92, 7)
        y = orc.conv(xs_o, ws, 1, 0, p)
        xs, tiles = s.share_packed(to_dev(x), stream_id=6)
        assert np.array_equal(to_np(xs), xs_o)
        wp = s.pack_weights_conv(to_dev(ws))
        check_consumers(s, p, y, (B, Co, H, W), lambda: s.conv1x1_product_prepacked(tiles, wp, B, C, H, W, Co), seed=92)
    for (M, K, N) in [(1, 2048, 1000), (5, 100, 9), (130, 4096, 65)]:
        say("dense product", n, t, hex(p), M, K, N)
        x = small_secrets((M, K), 5, bits, p)
        xs_o = orc.share(x, n, t, p, 92, 8)
        ws = orc.share(small_secrets((K, N), 6, bits - 2, p), n, t, p, 92, 9)
        y = orc.linear(xs_o, ws, p)
        xs, tiles = s.share_packed(to_dev(x), stream_id=8)
        wp = s.pack_weights_linear(to_dev(ws))
        check_consumers(s, p, y, (M, N, 1, 1), lambda: s.linear_product_prepacked(tiles, wp, M, K, N), seed=92)


# C, H, Co of 3 x 3 convolutions, five parties over the 61-bit prime
FULL_RANGE = [(512, 7, 96),     # tiles of 16 x 16, eight waves each, the contraction in two parts
              (512, 7, 128),    # tiles of 32 x 32, six runs
              (256, 14, 256),   # four runs
              (1024, 1, 401)]   # tiles of 64 x 64, every one shared by up to 15 workgroups: 16 planes, most of them zeros


@pytest.mark.parametrize("C,H,Co", FULL_RANGE)
def test_pending_product_full_range_operands_and_plane_sums(C, H, Co):
    """Uniform field elements as operands (what shares are), a contraction long enough that every tile has
    parts: the reduction of the pending product equals the reduction of the oracle's product."""
    n, t, p = 5, 2, binding.P61
    s = SSNet(n, t, f=13, seed=93)
    B, W, k = 1, H, 3
    xs, ws = field_uniform((n, B, C, H, W), 7), field_uniform((n, Co, C, k, k), 8)
    y = orc.conv(xs, ws, 1, 1, p)
    planes, wp = s.split_planes(to_dev(xs)), s.pack_weights_conv_taps(to_dev(ws))
    s.conv_product_planes(planes, wp, B, C, H, W, Co, k, k, 1, 1)
    out = torch.empty((n, B * Co * H * W), dtype=torch.int64, device="cuda")
    s.degree_reduce(None, stream_id=1, out=out)
    assert np.array_equal(to_np(out), orc.degree_reduce(y.reshape(n, -1), n, t, p, 93, 1))
    # repeated launches give the same bits (planes are rewritten in full every time)
    for i in range(20):
        s._ws[binding.WS_HEADER_BYTES:].fill_(1 + 7 * i)
        s.conv_product_planes(planes, wp, B, C, H, W, Co, k, k, 1, 1)
        again = torch.empty_like(out)
        s.degree_reduce(None, stream_id=1, out=again)
        assert bool(torch.equal(again, out))


def test_pending_product_errors():
    s = SSNet(5, 2, f=13, seed=1)
    out = torch.empty((5, 64), dtype=torch.int64, device="cuda")
    s.reserve(1 << 20)
    with pytest.raises(SSNetError) as ei:            # nothing pending
        s.degree_reduce(None, stream_id=0, out=out)
    assert ei.value.code == binding.EINVAL
    x = field_uniform((5, 1, 64, 4, 4), 1)
    w = field_uniform((5, 4, 64, 1, 1), 2)
    planes, wp = s.split_planes(to_dev(x)), s.pack_weights_conv_taps(to_dev(w))
    s.conv_product_planes(planes, wp, 1, 64, 4, 4, 4, 1, 1, 1, 0)      # 64 elements per party
    with pytest.raises(SSNetError) as ei:            # another element count than the pending product's
        s.degree_reduce(None, stream_id=0, out=torch.empty((5, 63), dtype=torch.int64, device="cuda"))
    assert ei.value.code == binding.EINVAL
    s.degree_reduce(None, stream_id=0, out=out)
    assert np.array_equal(to_np(out), orc.degree_reduce(orc.conv(x, w, 1, 0, binding.P61).reshape(5, -1), 5, 2, binding.P61, 1, 0))
    # a new workspace drops the pending product
    s._ws = None
    s.reserve(1 << 20)
    with pytest.raises(SSNetError) as ei:
        s.degree_reduce(None, stream_id=0, out=out)
    assert ei.value.code == binding.EINVAL


# (M, K, N) of a dense layer: two row tiles, the last one ragged; (B, C, H, W, Co, k, stride, pad) of a convolution
WHOLE_AHEAD = {(5, 2, binding.P61): ((101, 722, 3270), (3, 256, 32, 37, 128, 2, 1, 0)),
               (3, 1, binding.P61): ((101, 715, 5479), (3, 256, 36, 53, 128, 2, 1, 0)),
               (3, 1, binding.P45): ((99, 1968, 5487), (2, 256, 86, 67, 34, 3, 1, 0))}


@pytest.mark.parametrize("n,t,p", list(WHOLE_AHEAD))
def test_products_with_whole_tiles_ahead_of_the_cut_ones(n, t, p):
    """Tiles of 64 x 64 for two rounds of the chip and more: the first 256 lie in the first plane alone, the others in two.  Ragged rows
    and columns, columns that run over several images, and the same product as a tensor (the parts added up)."""
    s = SSNet(n, t, f=12, seed=94, p=p)
    bits = 11 if p == binding.P45 else 15
    (M, K, N), geom = WHOLE_AHEAD[n, t, p]
    assert s.lib.ssnet_product_bytes_linear(s._ctx, M, K, N) == 2 * 8 * n * M * N + 255 & ~255
    say("dense product, whole tiles first", n, t, hex(p), M, K, N)
    x = small_secrets((M, K), 5, bits, p)
    ws = orc.share(small_secrets((K, N), 6, bits - 2, p), n, t, p, 94, 9)
    y = orc.linear(orc.share(x, n, t, p, 94, 8), ws, p)
    _, tiles = s.share_packed(to_dev(x), stream_id=8)
    wp = s.pack_weights_linear(to_dev(ws))
    check_consumers(s, p, y, (M, N, 1, 1), lambda: s.linear_product_prepacked(tiles, wp, M, K, N), seed=94)
    assert np.array_equal(to_np(s.linear_mod_prepacked(tiles, wp, M, K, N)), y)
    say("conv product, whole tiles first", n, t, hex(p), geom)
    B, C, H, W, Co, k, stride, pad = geom
    xs = orc.share(small_secrets((B, C, H, W), 1, bits, p), n, t, p, 94, 5)
    ws = orc.share(small_secrets((Co, C, k, k), 2, bits - 2, p), n, t, p, 94, 6)
    y = orc.conv(xs, ws, stride, pad, p)
    planes, wp = s.split_planes(to_dev(xs)), s.pack_weights_conv_taps(to_dev(ws))
    geom = (B, C, H, W, Co, k, k, stride, pad)
    check_consumers(s, p, y, (B, Co) + y.shape[-2:], lambda: s.conv_product_planes(planes, wp, *geom), seed=94)
    assert np.array_equal(to_np(s.conv_mod_planes(planes, wp, *geom)), y)


# rows, contraction, columns: one, two, four and eight waves to a tile of 16 x 16, contractions in parts, either side the
# longer one, ragged edges on both, single blocks, contractions that leave waves without a unit
SMALL_DENSE = [(17, 64, 33), (1, 1, 1), (70, 250, 790), (64, 256, 128), (300, 130, 20), (20, 2400, 30), (16, 4096, 10), (9, 590, 16),
               (1, 400, 120), (129, 900, 48)]
SMALL_CONV = [  # B, C, H, W, Co, k, stride, pad
    (1, 512, 4, 4, 40, 3, 1, 1), (3, 64, 7, 5, 100, 1, 1, 0), (1, 64, 16, 15, 64, 3, 2, 1), (2, 128, 2, 2, 512, 3, 1, 1),
    (1, 192, 9, 9, 17, 5, 1, 2)]


@pytest.mark.parametrize("n,t,p", [(5, 2, binding.P61), (3, 1, binding.P45), (8, 3, binding.P61)])
def test_small_and_narrow_products(n, t, p):
    """Products whose tiles are computed by waves on their own: as tensors with full-range operands, and left to every
    consumer."""
    s = SSNet(n, t, f=12, seed=95, p=p)
    bits = 11 if p == binding.P45 else 15
    for i, (M, K, N) in enumerate(SMALL_DENSE):
        say("small dense", n, t, hex(p), M, K, N)
        x, w = (orc.share(small_secrets(sh, 2 * i + j, bits - 2 * j, p), n, t, p, 95, 8 + j) for j, sh in enumerate([(M, K), (K, N)]))
        y = orc.linear(x, w, p)
        assert np.array_equal(to_np(s.linear_mod(to_dev(x), to_dev(w))), y)
        _, tiles = s.share_packed(to_dev(small_secrets((M, K), 2 * i, bits, p)), stream_id=8)
        wp = s.pack_weights_linear(to_dev(w))
        check_consumers(s, p, y, (M, N, 1, 1), lambda: s.linear_product_prepacked(tiles, wp, M, K, N), seed=95)
        full_x, full_w = field_uniform((n, M, K), i) % np.uint64(p), field_uniform((n, K, N), 50 + i) % np.uint64(p)
        assert np.array_equal(to_np(s.linear_mod(to_dev(full_x), to_dev(full_w))), orc.linear(full_x, full_w, p))
    for (B, C, H, W, Co, k, stride, pad) in SMALL_CONV:
        say("small conv", n, t, hex(p), B, C, H, W, Co, k, stride, pad)
        xs = orc.share(small_secrets((B, C, H, W), 1, bits, p), n, t, p, 95, 5)
        ws = orc.share(small_secrets((Co, C, k, k), 2, bits - 2, p), n, t, p, 95, 6)
        y = orc.conv(xs, ws, stride, pad, p)
        planes, wp = s.split_planes(to_dev(xs)), s.pack_weights_conv_taps(to_dev(ws))
        geom = (B, C, H, W, Co, k, k, stride, pad)
        assert np.array_equal(to_np(s.conv_mod_planes(planes, wp, *geom)), y)
        check_consumers(s, p, y, (B, Co) + y.shape[-2:], lambda: s.conv_product_planes(planes, wp, *geom), seed=95)


def test_more_tiles_of_16_x_16_than_a_launch_holds():
    """One pixel of 128 channels under a 1 x 1 kernel, padded by 8192: a product of 1 x 268 million, zero but for the pixel."""
    import ctypes as Ct
    n, C, pad = 4, 128, 8192
    H = 1 + 2 * pad
    s = SSNet(n, 1, f=13, seed=5)
    xs, ws = field_uniform((n, 1, C, 1, 1), 1), field_uniform((n, 1, C, 1, 1), 2)
    planes, wp = s.split_planes(to_dev(xs)), s.pack_weights_conv_taps(to_dev(ws))
    geom = (1, C, 1, 1, 1, 1, 1, 1, pad)
    s.reserve(binding.WS_HEADER_BYTES + s.lib.ssnet_product_bytes_conv(s._ctx, *geom))
    out = torch.ones((n, H * H), dtype=torch.int64, device="cuda")
    assert s.lib.ssnet_conv_mod_planes(s._ctx, planes.data_ptr(), wp.data_ptr(), *geom, Ct.c_void_p(out.data_ptr())) == binding.OK
    centre = pad * H + pad
    assert np.array_equal(to_np(out[:, centre]), orc.conv(xs, ws, 1, 0, binding.P61).reshape(n))
    out[:, centre] = 0
    assert not any(bool(out[i].any()) for i in range(n))
    del out, s
    torch.cuda.empty_cache()


@pytest.mark.parametrize("p,N", [(binding.P61, 5472), (binding.P45, 7296)])
def test_second_operand_past_the_last_level(p, N):
    """16-row products on both sides of the 256 MB from which the second operand is read past the caches"""
    n, K, s = 3, 2048, SSNet(3, 1, f=12, seed=2, p=p)
    per = n * s.lib.ssnet_packed_weight_bytes(16, K)
    assert per * (N // 16 - 1) <= 256 << 20 < per * (N // 16)
    w = field_uniform((n, K, N), 1) % np.uint64(p)
    x = field_uniform((n, 3, K), 2) % np.uint64(p)
    want = orc.linear(x, w, p)
    for cols in (N - 16, N):
        say("last level", p, cols)
        wc = np.ascontiguousarray(w[:, :, :cols])
        got = s.linear_mod_packed(to_dev(x), s.pack_weights_linear(to_dev(wc)), cols)
        assert np.array_equal(to_np(got), want[:, :, :cols])


RAGGED = (7, 293, 890, 1351)   # n, M, K, N


def test_whole_tiles_stop_earlier_where_ragged_ones_shorten_the_ranges():
    """770 tiles with a ragged last column each: with 512 of them whole the ranges behind would be shorter than a full tile, and
    three of them could meet in one.  Workspace of two planes, the product as a tensor and through a reduction."""
    n, M, K, N = RAGGED
    s = SSNet(n, 3, f=12, seed=3)
    assert s.lib.ssnet_product_bytes_linear(s._ctx, M, K, N) == 2 * 8 * n * M * N + 255 & ~255
    x, w = field_uniform((n, M, K), 1), field_uniform((n, K, N), 2)
    y = orc.linear(x, w, binding.P61)
    d, wp = to_dev(x), s.pack_weights_linear(to_dev(w))
    assert np.array_equal(to_np(s.linear_mod_packed(d, wp, N)), y)
    tiles = s.pack_weights_linear(to_dev(np.ascontiguousarray(x.transpose(0, 2, 1))))   # the same tiles, rows as columns
    out = torch.empty((n, M, N), dtype=torch.int64, device="cuda")
    s.linear_product_prepacked(tiles, wp, M, K, N)
    s.degree_reduce(None, stream_id=3, out=out)
    assert np.array_equal(to_np(out), to_np(s.degree_reduce(to_dev(y), stream_id=3)))
