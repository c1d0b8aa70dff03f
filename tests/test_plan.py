"""The launch plan and the load kind at the edges of their rules (no GPU):
tests/plan_driver.cpp calls the library's plan_step and non_temporal_loads."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2502_11147_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(PKG, "libraas.so")):
        pytest.skip("needs g++ and the built library")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                           "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "plan_driver.cpp"), "-L", PKG,
                           "-l:libraas.so", "-Wl,-rpath," + PKG, "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                           "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", exe])

    def call(lines):
        res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return [tuple(int(x) for x in r.split()) for r in res.stdout.splitlines()]

    return call


def _plan(U, blocks, G=4, D=128, S=None, bf16=1, agg=0, npr=0, topk=8, cold=0, splits=0, page=16):
    nprb = npr * page // 32
    work = blocks + min(nprb, topk * max(1, page // 32))
    slots = S if S is not None else (blocks + nprb) * 32 // page
    lists = 4 + 6 * npr + npr * page // 32 if npr else 0
    return "plan %d %d %d %d %d %d %d %d %d %d %d %d" % (U, G, D, slots, blocks + nprb, work, bf16, agg, lists, splits,
                                                          npr, cold)


# (arguments, whether a unit is split): both sides of each line
SPLITS = [
    (dict(U=32, blocks=32), False), (dict(U=32, blocks=33), True),
    (dict(U=33, blocks=48), False), (dict(U=112, blocks=48), False), (dict(U=112, blocks=49), True),
    (dict(U=48, blocks=33, cold=1), True), (dict(U=49, blocks=39, cold=1), False), (dict(U=112, blocks=40, cold=1), True),
    (dict(U=113, blocks=64), False), (dict(U=113, blocks=65), True), (dict(U=128, blocks=65), True),
    (dict(U=129, blocks=256), False),
    (dict(U=16, blocks=40, G=8), False), (dict(U=16, blocks=41, G=8), True), (dict(U=17, blocks=48, G=8), False),
    (dict(U=8, blocks=48, G=16), False), (dict(U=64, blocks=48, G=16, cold=1), True), (dict(U=65, blocks=48, G=16, cold=1), False),
    (dict(U=16, blocks=48, G=7, D=64), False), (dict(U=64, blocks=48, G=7, D=64, cold=1), False),
    (dict(U=16, blocks=49, G=7, D=64), True),
    # 64 slots or fewer (page 64): as far as 64 blocks
    (dict(U=48, blocks=56, page=64), True), (dict(U=49, blocks=64, page=64), False), (dict(U=49, blocks=66, page=64), True),
    # fp32: half as many
    (dict(U=8, blocks=8, bf16=0), False), (dict(U=8, blocks=9, bf16=0), True), (dict(U=113, blocks=16, bf16=0), False),
    (dict(U=113, blocks=17, bf16=0), True),
    # prompt pages chosen by their own kernel
    (dict(U=32, blocks=32, agg=1, npr=256), True), (dict(U=64, blocks=32, agg=1, npr=256), False),
    (dict(U=8, blocks=32, agg=1, npr=1024), False), (dict(U=64, blocks=40, agg=1, npr=1536, cold=1), False),
    (dict(U=64, blocks=32, agg=1, npr=1664), True),  # (the slots' bounds no longer fit one workgroup's LDS)
]


@pytest.mark.parametrize("kw,split", SPLITS, ids=[",".join("%s=%s" % kv for kv in k.items()) for k, _ in SPLITS])
def test_split_rule(ask, kw, split):
    (waves, nsplit, _, _), = ask([_plan(**kw)])
    assert (nsplit > 1) == split and waves == (8 if kw["U"] <= 256 else 4)


def test_small_units_leave_the_fixed_array_alone(ask):
    """Whatever the plan does with units that one workgroup could cover, a
    static step keeps their scratch in the pool; forced splits use the array."""
    lines = [_plan(8, b, cold=c, G=g) for b in (33, 40, 48) for c in (0, 1) for g in (4, 16)]
    assert all(p[2] == 1 for p in ask(lines))
    assert [p[2] for p in ask([_plan(8, 49), _plan(8, 40, splits=3), _plan(8, 24, bf16=0, page=8),
                                 _plan(8, 25, bf16=0, page=8)])] == [0, 0, 1, 0]


def test_two_wavefronts_cover_their_unit(ask):
    """There are no split instances for workgroups of 2 wavefronts."""
    lines = [_plan(u, b, G=g, D=d, agg=a, npr=n, cold=c, page=p) for u in (1023, 1024, 5000) for b in (1, 8, 32, 33)
             for g in (1, 4, 7, 16) for d in (64, 128) for a in (0, 1) for n in (0, 64, 512, 1024) for c in (0, 1)
             for p in (16, 32)]
    plans = ask(lines)
    assert any(p[0] == 2 for p in plans)
    assert all(p[1] == 1 and p[3] == 1 for p in plans if p[0] == 2)


# units, bytes of the layer, bytes streamed since its last step, non-temporal loads
LOADS = [(256, 268e6, 0, 0), (256, 268e6, 268e6, 1), (104, 104e6, 104e6, 0), (104, 104e6, 208e6, 1),
         (128, 138e6, 138e6, 0), (128, 138e6, 276e6, 1), (256, 335e6, 0, 0), (256, 436e6, 0, 0), (256, 470e6, 0, 1),
         (512, 403e6, 0, 0), (384, 370e6, 0, 0), (384, 403e6, 0, 1), (1024, 537e6, 0, 1)]


@pytest.mark.parametrize("units,own,others,nt", LOADS)
def test_load_kind(ask, units, own, others, nt):
    assert ask(["loads %r %r %d 0" % (own, others, units)]) == [(nt,)]


@pytest.mark.parametrize("units,own,others,nt", [(64, 88e6, 176e6, 0), (64, 92e6, 184e6, 1), (256, 302e6, 0, 0),
                                                 (512, 352e6, 0, 1)])
def test_load_kind_with_a_prompt_region(ask, units, own, others, nt):
    assert ask(["loads %r %r %d 1" % (own, others, units)]) == [(nt,)]
