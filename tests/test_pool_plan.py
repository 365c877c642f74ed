"""How ReLU with pooling is cut into workgroups (csrc/pool_plan.hpp, the code that the launcher and the kernel use),
checked on the CPU over random geometries against what the two-launch form does: every input element opened by one
owner, every output pooled once, from rows that its workgroup keeps."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_02629_amd", "csrc")


class Rows(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("oh0", "oh1", "row0", "own1", "need1")]


class Plan(C.Structure):
    _fields_ = [("one_launch", C.c_bool)] + [(k, C.c_int) for k in ("P", "R", "strips", "threads")] + \
               [("blocks", C.c_size_t), ("lds", C.c_size_t)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool_plan")
    src = d / "pool_plan.cpp"
    src.write_text('#include "pool_plan.hpp"\nextern "C" {\n'
                   "ss_pool_rows cut(int s, int strips, int R, int H, int kh, int sh, int ph, int Ho)\n"
                   "{ return ss_pool_cut(s, strips, R, H, kh, sh, ph, Ho); }\n"
                   "ss_pool_plan plan(size_t planes, int H, int W, int kh, int sh, int Ho, bool out_in_mask)\n"
                   "{ return ss_plan_pool(planes, H, W, kh, sh, Ho, out_in_mask); }\n}\n")
    so = str(d / "pool_plan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(src)],
                   check=True)
    lib = C.CDLL(so)
    lib.cut.restype, lib.cut.argtypes = Rows, [C.c_int] * 8
    lib.plan.restype, lib.plan.argtypes = Plan, [C.c_size_t] + [C.c_int] * 5 + [C.c_bool]
    return lib


def geometries(count):
    rng = random.Random(5)
    while count:
        H, W = int(2 ** rng.uniform(0, 9)), int(2 ** rng.uniform(0, 11))
        kh, sh = rng.randint(1, min(9, H + 2)), rng.choice([1, 1, 2, 2, 3, 5, 9])
        ph = rng.randint(0, kh - 1)
        if kh > H + 2 * ph:
            continue
        count -= 1
        yield int(2 ** rng.uniform(0, 14)), H, W, kh, sh, ph, (H + 2 * ph - kh) // sh + 1


def test_every_element_has_one_owner_and_every_row_is_kept(lib):
    forms = set()
    for planes, H, W, kh, sh, ph, Ho in geometries(20000):
        p = lib.plan(planes, H, W, kh, sh, Ho, False)
        if not p.one_launch:
            forms.add("two launches")
            continue
        case = (planes, H, W, kh, sh, ph, Ho, p.P, p.R, p.strips)
        if p.strips == 1:
            forms.add("whole planes")
            assert p.blocks * p.P >= planes > (p.blocks - 1) * p.P and p.lds >= p.P * H * W * 8, case
            continue
        forms.add("strips")
        assert p.blocks == planes * p.strips and p.P == 1, case
        own, oh = 0, 0
        for s in range(p.strips):
            r = lib.cut(s, p.strips, p.R, H, kh, sh, ph, Ho)
            assert r.row0 == own and r.oh0 == oh and r.oh1 > r.oh0 and r.own1 >= r.row0, case
            own, oh = r.own1, r.oh1
            # rows that the kernels of this run meet: opened here, and inside its LDS
            lo, hi = max(0, r.oh0 * sh - ph), min(H, (r.oh1 - 1) * sh - ph + kh)
            assert r.row0 <= lo and r.need1 == hi and (hi - r.row0) * W * 8 <= p.lds <= 64 * 1024, case
        assert own == H and oh == Ho, case
    assert forms == {"two launches", "whole planes", "strips"}


def test_output_in_the_mask_goes_to_the_two_launches(lib):
    """In one launch, workgroups would write the output where others still read d_beta."""
    for planes, H, W, kh, sh, ph, Ho in geometries(5000):
        assert not lib.plan(planes, H, W, kh, sh, Ho, True).one_launch


def test_launches_hold_less_than_2_to_the_32_threads(lib):
    """Runs of less than their workgroup's threads: the two launches take one thread per element and still fit."""
    for planes, H, W, kh, sh, ph in [((1 << 24) - 1, 1, 129, 1, 1, 0), (1 << 24, 1, 129, 1, 1, 0), (1 << 24, 11, 20, 2, 2, 0),
                                     (1 << 21, 4, 300, 1, 1, 0), ((1 << 21) - 1, 4, 300, 1, 1, 0), (1 << 23, 2, 180, 1, 1, 0)]:
        assert planes * H * W < 1 << 32
        p = lib.plan(planes, H, W, kh, sh, (H + 2 * ph - kh) // sh + 1, False)
        assert p.one_launch == (p.blocks * p.threads < 1 << 32), (planes, H, W)
    assert not lib.plan(1 << 24, 1, 129, 1, 1, 1, False).one_launch
