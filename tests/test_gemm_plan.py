"""How a product is given to the kernels and cut into work (csrc/gemm_plan.hpp, the code that the launcher uses), checked on
the CPU over random shapes."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_02629_amd", "csrc")


class Plan(C.Structure):
    _fields_ = [("skinny", C.c_bool), ("ksplit", C.c_int), ("tiles", C.c_long), ("units", C.c_long)] + \
               [(k, C.c_int) for k in ("Kb", "G", "slots", "RT", "CT", "threads")] + \
               [(k, C.c_uint) for k in ("whole", "wlast", "tcost", "tlast", "cost", "cost0")]


def planner(directory, limbs):
    """plan(n, rows, cols, K, gather) of the library whose elements have `limbs` limbs; gather: 0 for operands in tiles, 1 for
    limb planes, their channels where a convolution reads them with a stride"""
    src = directory / "gemm_plan.cpp"
    src.write_text('#include "gemm_plan.hpp"\nextern "C" plan::gemm_plan plan_product(int n, int rows, int cols, int K, int gather)\n'
                   "{ return plan::plan_gemm(n, rows, cols, K, gather); }\n")
    so = str(directory / f"gemm_plan{limbs}.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-DSS_NS=plan", f"-DSS_NLIMB={limbs}", "-I", CSRC, "-o", so, str(src)], check=True)
    lib = C.CDLL(so)
    lib.plan_product.restype, lib.plan_product.argtypes = Plan, [C.c_int] * 5
    return lib.plan_product


@pytest.fixture(scope="module", params=[8, 6])
def plan(request, tmp_path_factory):
    return planner(tmp_path_factory.mktemp("gemm_plan"), request.param)


def test_launches_hold_less_than_2_to_the_32_threads(plan):
    """The runtime takes a larger grid without an error and runs a part of it.  Few rows and very many columns, as a convolution
    with a wide padding has them: the first two, 1 x 1 kernels over 128 channels of one pixel padded by 8192 and by 7327, have that
    many tiles of 16 x 16."""
    rng = random.Random(3)
    shapes = [(4, 1, 16385 ** 2, 128), (5, 1, 14655 ** 2, 128), (8, 15, 1 << 27, 384)]
    shapes += [(rng.randint(3, 8), int(2 ** rng.uniform(0, 20)), int(2 ** rng.uniform(16, 30)), 64 * rng.randint(1, 9)) for _ in range(50000)]
    for n, rows, cols, K in shapes:
        p = plan(n, rows, cols, K, 1)
        assert p.G * p.threads < 1 << 32 and (p.G >= 1 or p.tiles >= 1 << 30), (n, rows, cols, K, p.G, p.threads)
        assert p.threads == (256 if p.ksplit in (1, 2, 4) else 512)


# limbs and (n, rows, columns, contraction, gather) of products on either side of the line between the kernel of 16 x 16 tiles and the
# others, timed on an MI355X with weights from memory, product and reduction together: taken, 3 to 50 % faster; left, 5 to 30 % slower
TAKEN = [(8, (5, 128, 784, 512, 0)), (6, (3, 128, 784, 512, 0)), (8, (3, 1024, 196, 256, 0)), (8, (5, 1024, 196, 256, 0)), (8, (3, 256, 196, 1024, 0)),
         (8, (3, 1, 1000, 2048, 0)), (6, (3, 256, 196, 2304, 1)), (6, (3, 128, 784, 1152, 128)), (6, (4, 34, 192, 4608, 512)),
         (8, (3, 23, 968, 3200, 128)), (8, (5, 39, 726, 576, 64))]
LEFT = [(8, (5, 43, 578, 4608, 512)), (8, (3, 18, 1083, 12800, 512)), (8, (5, 270, 80, 4608, 512)), (6, (4, 27, 1152, 4608, 512)),
        (8, (5, 39, 1800, 4608, 1)), (8, (3, 94, 1352, 2304, 256)), (8, (5, 725, 75, 1375, 0)), (6, (5, 315, 579, 448, 0))]


def test_the_faster_kernel_on_both_sides_of_the_line(tmp_path):
    plans = {limbs: planner(tmp_path, limbs) for limbs in (8, 6)}
    for limbs, shape in TAKEN:
        assert plans[limbs](*shape).ksplit, (limbs, shape)
    for limbs, shape in LEFT:
        assert not plans[limbs](*shape).ksplit, (limbs, shape)


def test_planes_are_priced_by_what_a_unit_of_the_field_takes(tmp_path):
    """Over the 45-bit prime a unit takes 0.57 of the time and a plane as long as over the other: fewer tiles are worth cutting."""
    plans = {limbs: planner(tmp_path, limbs) for limbs in (8, 6)}
    for shape in [(5, 269, 579, 3245, 0), (3, 320, 1800, 576, 1), (4, 585, 310, 1010, 0)]:
        p = plans[6](*shape)
        assert p.slots == 1 and not p.ksplit and plans[8](*shape).slots > 1, shape
