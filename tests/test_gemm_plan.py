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


def product_planner(directory, limbs):
    """call(n, rows, cols, K, gather, tensor, room) -> (runs, workgroups, planes, plan_gemm's ksplit, slots, whole): what the launcher takes.
    runs > 0: gemm_square_kernel, else plan_gemm's kernel.  tensor: the planes are added up; room: planes that there is memory for."""
    src = directory / "product_plan.cpp"
    src.write_text('#include "gemm_plan.hpp"\nextern "C" void plan_product(int n, int rows, int cols, int K, int gather, int tensor, int room, long *v)\n'
                   "{ const plan::product_plan r = plan::plan_product(n, rows, cols, K, gather, tensor, room);\n"
                   "  const long w[6] = {r.sq.runs, (long)r.sq.G, r.planes(), r.p.ksplit, r.p.slots, (long)r.p.whole};\n"
                   "  for (int i = 0; i < 6; i++) v[i] = w[i]; }\n")
    so = str(directory / f"product_plan{limbs}.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-DSS_NS=plan", f"-DSS_NLIMB={limbs}", "-I", CSRC,
                    "-o", so, str(src)], check=True)
    fn = C.CDLL(so).plan_product
    fn.restype, fn.argtypes = None, [C.c_int] * 7 + [C.POINTER(C.c_long)]

    def call(n, rows, cols, K, gather, tensor, room):
        v = (C.c_long * 6)()
        fn(n, rows, cols, K, gather, tensor, room, v)
        return tuple(v)
    return call


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
        (8, (5, 39, 1800, 4608, 1)), (8, (3, 94, 1352, 2304, 256)), (8, (4, 46, 720, 4608, 1)), (6, (5, 315, 579, 448, 0)),
        (6, (5, 144, 361, 6400, 1)), (6, (5, 43, 847, 6400, 1)), (8, (4, 71, 408, 4397, 0))]


def test_the_faster_kernel_on_both_sides_of_the_line(tmp_path):
    plans = {limbs: planner(tmp_path, limbs) for limbs in (8, 6)}
    for limbs, shape in TAKEN:
        assert plans[limbs](*shape).ksplit, (limbs, shape)
    for limbs, shape in LEFT:
        assert not plans[limbs](*shape).ksplit, (limbs, shape)


def test_planes_are_priced_by_what_a_unit_of_the_field_takes(tmp_path):
    """Over the 45-bit prime a unit takes 0.57 of the time and a plane as long as over the other: fewer tiles are worth cutting."""
    plans = {limbs: planner(tmp_path, limbs) for limbs in (8, 6)}
    for shape in [(5, 269, 579, 3245, 0), (3, 320, 1800, 576, 1), (4, 52, 3468, 1152, 1)]:
        p = plans[6](*shape)
        assert p.slots == 1 and not p.ksplit and plans[8](*shape).slots > 1, shape


def test_products_of_the_gpu_tests_take_what_these_are_written_for(tmp_path):
    """Kernel, planes and whole tiles ahead of each product of tests/test_gpu_pending_product.py, left in the workspace and as a tensor.
    A change of the rules that moves one of them asks for another shape there."""
    import test_gpu_pending_product as g
    plans = {limbs: product_planner(tmp_path, limbs) for limbs in (8, 6)}
    limbs_of = {g.binding.P61: 8, g.binding.P45: 6}

    def taken(limbs, *shape):
        """of the pending product: ("square", runs), ("waves", waves of a tile, planes) or ("tiles", planes, whole tiles ahead)"""
        def one(tensor, room):
            runs, _, planes, ksplit, _, whole = plans[limbs](*shape, tensor, room)
            return ("square", runs) if runs else ("waves", ksplit, planes) if ksplit else ("tiles", planes, whole)
        pending, tensor = one(0, 8), one(1, 0)
        if pending[0] == "tiles":   # the tests of tiles of 64 x 64 run both forms
            assert tensor == pending, (limbs, shape, pending, tensor)
        return pending

    def conv(limbs, n, B, C, H, W, Co, k, stride, pad):
        Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
        return taken(limbs, n, Co, B * Ho * Wo, C * k * k, C if stride > 1 else 1)

    assert [conv(8, 5, *c) for c in g.CONV_CASES[:6]] == [("square", 4), ("square", 1), ("waves", 2, 1), ("square", 6), ("square", 6), ("waves", 4, 1)]
    assert [conv(8, 3, *g.CONV_CASES[i]) for i in (0, 3, 4)] == [("square", 3), ("square", 8), ("square", 6)]
    assert [conv(8, 7, *g.CONV_CASES[i]) for i in (0, 3, 4)] == [("tiles", 4, 0), ("square", 8), ("square", 6)]
    assert [conv(6, 5, *g.CONV_CASES[i]) for i in (0, 3, 4, 6)] == [("square", 3), ("square", 6), ("waves", 4, 1), ("square", 5)]
    assert {key: [conv(limbs_of[key[2]], key[0], *c) for c in cases] for key, cases in g.CUT_TILES.items()} == {
        (5, 2, g.binding.P61): [("tiles", 16, 0), ("tiles", 5, 0)], (3, 1, g.binding.P61): [("tiles", 14, 0)],
        (7, 3, g.binding.P61): [("tiles", 5, 0)], (5, 2, g.binding.P45): [("tiles", 12, 0)]}
    assert [conv(8, 5, 1, C, H, H, Co, 3, 1, 1) for C, H, Co in g.FULL_RANGE] == [("waves", 8, 2), ("square", 6), ("square", 4), ("tiles", 16, 0)]
    for (n, t, p), ((M, K, N), c) in g.WHOLE_AHEAD.items():
        assert taken(limbs_of[p], n, M, N, K, 0) == conv(limbs_of[p], n, *c) == ("tiles", 2, 256)
    n, M, K, N = g.RAGGED
    assert taken(8, n, M, N, K, 0) == ("tiles", 2, 256) and planner(tmp_path, 8)(n, M, N, K, 0).tiles >= 3 * 256
    # one, two, four and eight waves, and a contraction in parts
    small = [taken(limbs, n, M, N, K, 0) for limbs, n in ((8, 5), (6, 3), (8, 8)) for M, K, N in g.SMALL_DENSE]
    small += [conv(limbs, n, *c) for limbs, n in ((8, 5), (6, 3), (8, 8)) for c in g.SMALL_CONV]
    waves = [s[1:] for s in small if s[0] == "waves"]
    assert {k for k, _ in waves} == {1, 2, 4, 8} and max(planes for _, planes in waves) > 1
