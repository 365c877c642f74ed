"""Small products whose column operand reaches the product kernel as field elements (product_plan::element_waves in
csrc/gemm_plan.hpp, gemm_ksplit_kernel), and dense layers whose two operands are packed in one launch."""
import ctypes as C
import subprocess

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2406_02629_amd import SSNet, binding
from test_gemm_plan import CSRC
from util import field_uniform, to_dev, to_np

P61, P45 = binding.P61, binding.P45

# (M, K, N) of a dense layer, (B, C, H, W, Co, k, stride, pad) of a convolution -> waves that share a tile, three parties: rows and
# columns of one element, full and ragged blocks, contractions of one k block to eight, one element past them, kernels wider than their
# padding, strides, several images in a block of pixels
SMALL = {(1, 1, 1): 1, (1, 64, 16): 1, (16, 65, 17): 2, (17, 63, 130): 1, (3, 128, 33): 2, (5, 129, 10): 4, (40, 256, 31): 4, (1, 257, 120): 8,
         (300, 1, 300): 1, (8, 512, 100): 8, (9, 500, 49): 8, (33, 130, 47): 4, (2, 400, 120): 8,
         (1, 1, 28, 28, 6, 5, 1, 2): 1, (1, 6, 14, 14, 16, 5, 1, 0): 4, (3, 3, 9, 7, 33, 3, 2, 1): 1, (2, 70, 5, 5, 17, 1, 1, 0): 2, (1, 20, 6, 11, 50, 5, 1, 2): 8,
         (2, 2, 4, 4, 2, 4, 1, 0): 1, (5, 3, 3, 3, 20, 3, 1, 2): 1, (1, 128, 1, 1, 30, 2, 3, 1): 8, (1, 3, 20, 20, 16, 7, 2, 3): 4}
# left to a launch that packs: longer contractions, more tiles than run at a time, wide rows (0), and operands packed together
PACKED = [(20, 513, 40), (16, 512, 1000), (200, 300, 500), (33, 700, 129), (1, 2100, 300), (260, 640, 700)]


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    """waves[limbs](n, rows, cols, K, input_rows)"""
    directory = tmp_path_factory.mktemp("element_plan")
    src = directory / "plan.cpp"
    src.write_text('#include "gemm_plan.hpp"\nextern "C" int waves(int n, int rows, int cols, int K, int input_rows, long *G)\n'
                   "{ const plan::product_plan r = plan::plan_product(n, rows, cols, K, 0, true, 0);\n"
                   "  const int w = r.element_waves(input_rows); if (w) *G = r.for_elements(w).p.G; return w; }\n")
    out = {}
    for limbs in (8, 6):
        so = str(directory / f"plan{limbs}.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-DSS_NS=plan", f"-DSS_NLIMB={limbs}", "-I", CSRC,
                        "-o", so, str(src)], check=True)
        fn = C.CDLL(so).waves
        fn.restype, fn.argtypes = C.c_int, [C.c_int] * 5 + [C.POINTER(C.c_long)]
        out[limbs] = fn
    return out


def test_which_products_take_elements(waves):
    G = C.c_long()
    for limbs in (8, 6):
        for shape, want in SMALL.items():
            if len(shape) == 3:
                M, K, N = shape
                got = waves[limbs](3, M, N, K, M, C.byref(G))
                tiles = 3 * (-(-M // 16)) * (-(-N // 16))
            else:
                B, Ci, H, W, Co, k, stride, pad = shape
                cols, K = B * ((H + 2 * pad - k) // stride + 1) * ((W + 2 * pad - k) // stride + 1), Ci * k * k
                got = waves[limbs](3, Co, cols, K, 0, C.byref(G))
                tiles = 3 * (-(-Co // 16)) * (-(-cols // 16))
            assert got == want and got >= -(-K // 64) and tiles * got <= 2048, (limbs, shape, got)
            assert G.value == (tiles if got == 8 else -(-tiles // (4 // got))), (limbs, shape)
        for M, K, N in PACKED:
            assert waves[limbs](3, M, N, K, M, C.byref(G)) == 0, (limbs, M, K, N)


@pytest.mark.gpu
@pytest.mark.parametrize("n,t,p", [(3, 1, P61), (3, 1, P45), (8, 3, P61)])
def test_products_of_elements(n, t, p):
    s = SSNet(n, t, f=12, seed=97, p=p)
    for shape in list(SMALL) + PACKED:
        print("elements", n, hex(p), shape, flush=True)
        if len(shape) == 3:
            M, K, N = shape
            x, w = (field_uniform((n,) + sh, i) % np.uint64(p) for i, sh in enumerate(((M, K), (K, N))))
            want = orc.linear(x, w, p)
            assert np.array_equal(to_np(s.linear_mod(to_dev(x), to_dev(w))), want)
            assert np.array_equal(to_np(s.linear_mod_packed(to_dev(x), s.pack_weights_linear(to_dev(w)), N)), want)
        else:
            B, Ci, H, W, Co, k, stride, pad = shape
            x, w = (field_uniform((n,) + sh, i) % np.uint64(p) for i, sh in enumerate(((B, Ci, H, W), (Co, Ci, k, k))))
            got = s.conv_mod_packed(to_dev(x), s.pack_weights_conv(to_dev(w)), Co, k, k, stride, pad)
            assert np.array_equal(to_np(got), orc.conv(x, w, stride, pad, p))


# (M, K = N) and (B, C = Co, H, W, k, pad): the output has the size of the input, and lies in its memory or reaches into it
IN_PLACE = [(8, 512), (40, 31), (1, 257), (200, 64), (2, 6, 14, 14, 3, 1), (1, 40, 9, 7, 1, 0), (3, 2, 5, 5, 5, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", IN_PLACE)
def test_output_in_the_memory_of_the_input(shape):
    """Other workgroups read the input after the first ones have stored their outputs: the input is packed first, as for every larger product."""
    n, dense = 3, len(shape) == 2
    s = SSNet(n, 1, f=12, seed=97)
    xshape = (n,) + (shape if dense else shape[:4])
    wshape = (n, shape[1], shape[1]) if dense else (n, shape[1], shape[1], shape[4], shape[4])
    x, w = field_uniform(xshape, 1), field_uniform(wshape, 2)
    want = orc.linear(x, w, P61) if dense else orc.conv(x, w, 1, shape[5], P61)
    wp = s.pack_weights_linear(to_dev(w)) if dense else s.pack_weights_conv(to_dev(w))

    def product(src, dst):
        if dense:
            return s.linear_mod_packed(src, wp, shape[1], out=dst)
        return s.conv_mod_packed(src, wp, shape[1], shape[4], shape[4], 1, shape[5], out=dst)

    count = x.size
    for shift in (0, 1, -1, count - 1, 1 - count, count, -count):   # elements from the input's start to the output's
        print("in place", shape, shift, flush=True)
        memory = torch.zeros(3 * count, dtype=torch.int64, device="cuda")
        src, dst = (memory[at:at + count].view(xshape) for at in (count, count + shift))
        src.copy_(to_dev(x))
        s.profile_begin()
        assert np.array_equal(to_np(product(src, dst)), want), shift
        assert s.profile_end()["pack_x"][1] == (abs(shift) < count), shift
    if dense:
        src = to_dev(x)
        assert np.array_equal(to_np(s.linear_mod(src, to_dev(w), out=src)), want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,pack_w,pack_x", [((40, 256, 31), 1, 0), ((33, 700, 129), 0, 1)])
def test_profile_classes_of_a_fresh_dense_layer(shape, pack_w, pack_x):
    """weights alone where the input is read as field elements, else both operands in one launch: include/ssnet.h at ssnet_profile_begin"""
    M, K, N = shape
    s = SSNet(3, 1, f=12, seed=97)
    x, w = to_dev(field_uniform((3, M, K), 1)), to_dev(field_uniform((3, K, N), 2))
    s.linear_mod(x, w)
    s.profile_begin()
    s.linear_mod(x, w)
    spans = {name: count for name, (_, count) in s.profile_end().items()}
    assert (spans["pack_w"], spans["pack_x"], spans["gemm"]) == (pack_w, pack_x, 1)
