"""Products on gemm_square_kernel (tiles of 32 x 32, the contraction in runs with a plane each) and the rule that takes them there
(csrc/gemm_plan.hpp: plan_product, of which plan_gemm is what a product falls back to)."""
import random

import numpy as np
import pytest
import torch

import oracle as orc
import test_gpu_pending_product as pending
from paper_2406_02629_amd import SSNet, binding
from test_gemm_plan import product_planner
from util import field_uniform, to_dev, to_np

P61, P45 = binding.P61, binding.P45

# per scheme and field: (M, K, N) of dense layers, (B, C, H, W, Co, k, stride, pad) of convolutions on limb planes -> runs of the
# pending product, runs of the product as a tensor (0: another kernel).  Odd and even numbers of blocks on either side, the last one
# with one row or column or full, runs of unequal length, one run to eight.
SHAPES = {
    (5, 2, P61): {(18, 139, 1642): (1, 1), (18, 494, 545): (2, 0), (17, 520, 413): (3, 0), (33, 1043, 186): (4, 0), (243, 858, 18): (5, 0),
                  (17, 1032, 17): (6, 0), (17, 1447, 17): (8, 0), (164, 2174, 33): (4, 4),
                  (3, 192, 28, 23, 18, 1, 1, 0): (1, 1), (2, 128, 7, 7, 200, 3, 1, 0): (3, 3), (1, 128, 13, 5, 182, 3, 1, 0): (4, 0),
                  (3, 64, 5, 13, 18, 5, 1, 0): (7, 0), (1, 64, 9, 19, 200, 3, 2, 1): (3, 0), (1, 512, 4, 11, 163, 2, 2, 1): (8, 0)},
    (3, 1, P45): {(156, 66, 1942): (1, 1), (17, 404, 1808): (2, 1), (18, 688, 712): (3, 0), (17, 1579, 17): (5, 0), (17, 1974, 21): (8, 0),
                  (3, 64, 28, 28, 230, 1, 1, 0): (1, 1), (1, 64, 23, 5, 35, 5, 1, 0): (5, 0), (3, 192, 13, 3, 204, 3, 1, 0): (6, 0),
                  (3, 512, 29, 27, 51, 1, 2, 0): (2, 0), (1, 64, 8, 18, 17, 5, 2, 2): (5, 0)},
    (7, 3, P61): {(33, 1071, 229): (2, 2), (1, 128, 12, 3, 98, 3, 1, 1): (4, 0)},
}
# products that stay with tiles of 64 x 64 -> how they are cut when left in the workspace, and as a tensor: several planes, whole tiles alone, and
# whole tiles ahead of cut ones ("square": the tensor is a product in runs)
OTHERS = {
    (5, 2, P61): {(819, 1558, 8): ("planes", "planes"), (33, 693, 7634): ("ahead", "ahead"), (3, 192, 99, 87, 40, 2, 2, 1): ("ahead", "ahead")},
    (3, 1, P61): {(36, 521, 5092): ("whole", "whole"), (3, 192, 27, 94, 328, 2, 2, 0): ("ahead", "ahead")},
    (7, 3, P61): {(39, 516, 5766): ("ahead", "square"), (33, 636, 5309): ("ahead", "ahead"), (2, 512, 2, 2, 578, 3, 1, 1): ("planes", "planes"),
                  (1, 64, 25, 105, 100, 3, 1, 1): ("ahead", "square")},
    (5, 2, P45): {(33, 928, 6914): ("ahead", "square"), (34, 1448, 6620): ("ahead", "ahead"), (908, 1931, 34): ("planes", "planes"),
                  (1, 512, 3, 3, 842, 3, 1, 1): ("planes", "planes"), (3, 192, 16, 76, 426, 3, 2, 1): ("ahead", "ahead")},
}


def product_of(shape):
    """rows, columns, contraction and gather of the product of a dense layer or a convolution"""
    if len(shape) == 3:
        return shape[0], shape[2], shape[1], 0
    B, Ci, H, W, Co, k, stride, pad = shape
    cols = B * ((H + 2 * pad - k) // stride + 1) * ((W + 2 * pad - k) // stride + 1)
    return Co, cols, Ci * k * k, Ci if stride > 1 else 1


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans[limbs](n, rows, cols, K, gather, tensor, room) -> (runs, workgroups, planes, plan_gemm's ksplit, slots, whole)"""
    directory = tmp_path_factory.mktemp("square_plan")
    return {limbs: product_planner(directory, limbs) for limbs in (8, 6)}


def test_shapes_of_the_gpu_tests_take_what_they_are_written_for(plans):
    for (n, t, p), shapes in SHAPES.items():
        for shape, runs in shapes.items():
            product = product_of(shape)
            call = plans[8 if p == P61 else 6]
            assert (call(n, *product, 0, 8)[0], call(n, *product, 1, 0)[0]) == runs, (n, shape)
    for (n, t, p), shapes in OTHERS.items():
        for shape, kinds in shapes.items():
            for kind, (tensor, room) in zip(kinds, ((0, 8), (1, 0))):
                runs, _, planes, ksplit, slots, whole = plans[8 if p == P61 else 6](n, *product_of(shape), tensor, room)
                assert (runs > 0) == (kind == "square") and ksplit == 0, (n, shape, tensor)
                if runs == 0:
                    assert planes == slots, (n, shape, tensor)
                    assert {"planes": slots >= 5, "whole": slots == 1 and whole > 0, "ahead": slots == 2 and whole >= 256}[kind], (n, shape, tensor)


# limbs, (n, rows, columns, contraction, gather) -> runs of the pending product, as the comment at plan_square has them: faster there, and left (0) to
# tiles of 64 x 64 and to waves on their own, which are faster
TIMED = {(8, (5, 128, 784, 1152, 1)): 1, (8, (5, 128, 784, 1152, 128)): 1, (8, (5, 256, 196, 1024, 0)): 4, (8, (5, 512, 49, 2048, 0)): 3,
         (8, (5, 256, 196, 2304, 1)): 4, (8, (5, 512, 49, 4608, 1)): 3, (8, (3, 128, 1024, 1152, 1)): 2, (6, (3, 512, 49, 4608, 1)): 5, (6, (3, 256, 196, 2304, 1)): 3,
         (8, (5, 64, 3136, 576, 1)): 0, (8, (3, 690, 441, 576, 1)): 0, (8, (7, 203, 576, 500, 0)): 0, (8, (3, 66, 256, 6400, 1)): 0,
         (8, (3, 384, 338, 2304, 1)): 0, (8, (5, 128, 6272, 1152, 1)): 0, (8, (5, 256, 1568, 1024, 0)): 0, (8, (5, 256, 1568, 1024, 1)): 0, (8, (3, 895, 8712, 3200, 1)): 0,
         (8, (5, 512, 49, 4608, 512)): 3, (8, (5, 256, 392, 1152, 128)): 3, (8, (3, 196, 196, 1600, 1)): 5, (6, (3, 256, 676, 3456, 1)): 3}   # (the last row: taken and slower)


def test_timed_products_take_what_their_comment_says(plans):
    for (limbs, product), runs in TIMED.items():
        assert plans[limbs](*product, 0, 8)[0] == runs, (limbs, product)


def test_planes_stay_within_the_room_and_workgroups_within_a_launch(plans):
    rng = random.Random(11)
    taken = 0
    for _ in range(20000):
        limbs, n, gather = rng.choice([8, 6]), rng.randint(3, 8), rng.choice([0, 1, 64, 512])
        rows, cols = int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 24))
        K = 64 * rng.randint(1, 150) if gather else rng.randint(1, 9600)
        for tensor, room in ((0, 8), (0, 0), (0, rng.randint(1, 8)), (1, 0)):
            runs, G, planes, _, slots, _ = plans[limbs](n, rows, cols, K, gather, tensor, room)
            assert planes <= max(slots, 0 if tensor else room), (limbs, n, rows, cols, K, gather, tensor, room)
            if runs:
                taken += 1
                Rb, Cb = -(-rows // 16), -(-cols // 16)
                assert 1 <= runs <= min(8, -(-K // 64)) and 2 <= Rb < 1 << 16 and 2 <= Cb < 1 << 16
                assert G == n * ((Rb + 1) // 2) * ((Cb + 1) // 2) * runs < 1 << 24
    assert taken > 10000


def operands(s, n, t, p, shape, full):
    """x, w as shares of small values, or full-range field elements"""
    xshape, wshape = (shape[:2], shape[1:]) if len(shape) == 3 else (shape[:4], (shape[4], shape[1], shape[5], shape[5]))
    if full:
        return field_uniform((n,) + xshape, 3) % np.uint64(p), field_uniform((n,) + wshape, 4) % np.uint64(p)
    bits = 11 if p == P45 else 15
    return (orc.share(pending.small_secrets(sh, i, bits - 2 * i, p), n, t, p, 96, 5 + i) for i, sh in enumerate((xshape, wshape)))


def run_shape(s, n, t, p, shape):
    """as a tensor with full-range operands, and left to every consumer"""
    pending.say("product", n, t, hex(p), shape)
    if len(shape) == 3:
        M, K, N = shape
        x, w = operands(s, n, t, p, shape, True)
        assert np.array_equal(to_np(s.linear_mod(to_dev(x), to_dev(w))), orc.linear(x, w, p))
        x, w = operands(s, n, t, p, shape, False)
        tiles, wp = s.pack_weights_linear(to_dev(np.ascontiguousarray(x.transpose(0, 2, 1)))), s.pack_weights_linear(to_dev(w))
        pending.check_consumers(s, p, orc.linear(x, w, p), (M, N, 1, 1), lambda: s.linear_product_prepacked(tiles, wp, M, K, N), seed=96)
        return
    B, Ci, H, W, Co, k, stride, pad = shape
    geom = (B, Ci, H, W, Co, k, k, stride, pad)
    x, w = operands(s, n, t, p, shape, True)
    planes, wp = s.split_planes(to_dev(x)), s.pack_weights_conv_taps(to_dev(w))
    assert np.array_equal(to_np(s.conv_mod_planes(planes, wp, *geom)), orc.conv(x, w, stride, pad, p))
    x, w = operands(s, n, t, p, shape, False)
    y = orc.conv(x, w, stride, pad, p)
    planes, wp = s.split_planes(to_dev(x)), s.pack_weights_conv_taps(to_dev(w))
    pending.check_consumers(s, p, y, (B, Co) + y.shape[-2:], lambda: s.conv_product_planes(planes, wp, *geom), seed=96)


@pytest.mark.gpu
@pytest.mark.parametrize("n,t,p", list({**SHAPES, **OTHERS}))
def test_products_in_runs_and_in_tiles_of_64(n, t, p):
    s = SSNet(n, t, f=12, seed=96, p=p)
    for shape in list(SHAPES.get((n, t, p), ())) + list(OTHERS.get((n, t, p), ())):
        run_shape(s, n, t, p, shape)


@pytest.mark.gpu
def test_a_workspace_without_room_for_further_planes():
    """Three runs where there is room for their planes behind the messages of every consumer, else plan_gemm's kernel with its one plane in the
    room that this needs; less is refused."""
    (M, K, N), n, t = (17, 520, 413), 5, 2
    s = SSNet(n, t, f=12, seed=96)
    x, w = operands(s, n, t, P61, (M, K, N), True)
    tiles, wp = s.pack_weights_linear(to_dev(np.ascontiguousarray(x.transpose(0, 2, 1)))), s.pack_weights_linear(to_dev(w))
    want = orc.degree_reduce(orc.linear(x, w, P61).reshape(n, -1), n, t, P61, 96, 3)
    plane = 8 * n * M * N
    assert s.lib.ssnet_product_bytes_linear(s._ctx, M, K, N) == 3 * plane + 255 & ~255
    out = torch.empty((n, M, N), dtype=torch.int64, device="cuda")
    reduce_bytes = 8 * (5 * 3 + 3 * n) * M * N
    for extra, code in ((1 << 20, binding.OK), (512, binding.OK), (-4096, binding.EWORKSPACE)):
        ws = torch.zeros(binding.WS_HEADER_BYTES + reduce_bytes + plane + extra, dtype=torch.uint8, device="cuda")
        assert s.lib.ssnet_set_workspace(s._ctx, ws.data_ptr(), ws.numel()) == binding.OK
        assert s.lib.ssnet_linear_product_prepacked(s._ctx, tiles.data_ptr(), wp.data_ptr(), M, K, N) == binding.OK
        assert s.lib.ssnet_degree_reduce(s._ctx, None, M * N, 3, out.data_ptr()) == code, extra
        if code == binding.OK:
            assert np.array_equal(to_np(out).reshape(n, -1), want)
