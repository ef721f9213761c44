"""The stream-K GEMM schedule's arithmetic, modelled on the host.

The kernels (gemm.hip: sk_plan, sk_range, sk_owner, sk_next_item and gemm_fix's contributor
walk) split T tiles of nk K steps over P workgroups: whole data-parallel units first, then a
stream-K tail over the first Pk workgroups, whose range cuts leave fp32 partial tiles that the fixup
adds.  This model restates those formulas (schedule_model.py) and checks, for fixed and random (T, P, nk),
that every (tile, K step) is computed exactly once, that every partial slot is written once and read by
exactly the fixup of its tile, and that the fixup's pieces of a tile cover K in order.  The whole-tile rules
(a short K with fewer tiles than workgroups, one wave at least 7/8 full, whole waves when the last one is
full or at least half full) give an empty tail.  The bf16 projections choose their tile by estimates that
the model restates too; the shapes of the GPU tests are checked to reach the plans they are there for.
"""
import os
import random
import re

import pytest

import schedule_model as M
from paper_2606_13898_amd import build
from schedule_model import cut_plan, plan, whole_tiles


def test_model_holds_the_kernels_constants():
    with open(os.path.join(build.CSRC, "gemm.hip")) as f:
        src = f.read()
    with open(os.path.join(build.CSRC, "kernels.h")) as f:
        assert f"kGemmWorkgroups = {M.WORKGROUPS};" in f.read()
    assert f"kNoSplitSteps = {M.NO_SPLIT_STEPS};" in src and f"kSkMinSteps = {M.MIN_STEPS};" in src
    for tile, costs in M.TILE_COSTS.items():
        assert re.search(rf"plan_cost<EPI>\(r{tile} \* .*, nk, TileCost\{{{', '.join(map(str, costs))}\}}\);", src), tile
    assert f"(EPI == EPI_RESID ? {M.LAUNCH_Z} : {M.LAUNCH});" in src
    assert "turns * ((nk + 3) / 4 * (tiles <= P ? {} : {}) + {}) < best".format(*M.SMALL_COSTS) in src


def rng(I, P, w):
    return I * w // P, I * (w + 1) // P


def owner(I, P, a):
    return ((a + 1) * P - 1) // I


def check(T, P, nk, plan=plan):
    s, U, dp, ln, I, Pk = plan(T, P, nk)
    ln = max(ln, 1)
    cover, slots, direct = {}, {}, set()
    for pid in range(P):
        u = pid
        b, e = rng(I, Pk, pid) if pid < Pk else (I, I)
        it = b
        while True:
            if u < dp:
                pc, t = divmod(u, T)
                kb, ke = pc * nk // s, (pc + 1) * nk // s
                slot = None if s == 1 else u
                u += P
            elif it < e:
                v = it // ln
                k0 = it - v * ln
                k1 = min(ln, k0 + e - it)
                pc, t = divmod(dp + v, T)
                base = pc * nk // s
                kb, ke = base + k0, base + k1
                whole = s == 1 and k0 == 0 and k1 == ln
                slot = None if whole else P + 2 * pid + (0 if it == b else 1)
                it += k1 - k0
            else:
                break
            assert 0 <= kb < ke <= nk
            for k in range(kb, ke):
                assert (t, k) not in cover
                cover[(t, k)] = pid
            if slot is None:
                direct.add(t)
            else:
                assert slot not in slots and slot < 3 * P
                slots[slot] = (t, kb, ke)
    assert len(cover) == T * nk
    read, fixed = set(), set()
    for f in range(T if s > 1 else U - dp):
        t = f if s > 1 else dp + f
        got, skip = [], False
        for pc in range(s):
            u = pc * T + t
            if u < dp:
                got.append(u)
                continue
            a0 = (u - dp) * ln
            w0, w1 = owner(I, Pk, a0), owner(I, Pk, a0 + ln - 1)
            if s == 1 and w0 == w1:
                skip = True
                break
            for w in range(w0, w1 + 1):
                b, e = rng(I, Pk, w)
                if b < e:
                    got.append(P + 2 * w + (0 if b // ln == u - dp else 1))
        if skip:
            assert t in direct
            continue
        ks = []
        for sl in got:
            assert sl in slots and slots[sl][0] == t and sl not in read
            read.add(sl)
            ks.append(slots[sl][1:])
        ks.sort()
        assert ks[0][0] == 0 and ks[-1][1] == nk
        assert all(ks[i][1] == ks[i + 1][0] for i in range(len(ks) - 1))
        assert t not in direct
        fixed.add(t)
    assert read == set(slots)
    assert fixed | direct == set(range(T)) and not (fixed & direct)


@pytest.mark.parametrize("T,P,nk", [(528, 256, 48), (396, 256, 48), (132, 256, 192), (1, 256, 128),
                                    (257, 256, 5), (3, 7, 100), (0, 256, 4), (100, 256, 65), (256, 256, 192),
                                    (512, 256, 3), (384, 256, 48), (383, 256, 48)])
def test_schedule_fixed_cases(T, P, nk):
    check(T, P, nk)
    check(T, P, nk, cut_plan)


def test_short_tail_goes_to_fewer_workgroups():
    # 528 tiles on 256 workgroups: two whole waves, then 16 tiles x 48 steps over 64 workgroups
    assert not whole_tiles(528, 256, 48)
    s, U, dp, ln, I, Pk = plan(528, 256, 48)
    assert (s, dp, ln, I, Pk) == (1, 512, 48, 768, 64)


def test_projections_at_the_64x64_workload():
    # 2254 image rows (12 row tiles of 192) + 512 text rows (3), D = 3072, F = 12288: all four on 192 x 192;
    # QKV 720 tiles and MLP up 960 run whole waves (3 and 4, the last 208 and 192 tiles), the attention output
    # and MLP down 240 tiles in one wave (more than 7/8 full)
    assert M.projections([(2254, 512)], 3072, 12288) == dict(
        qkv=(192, 720, 1, 720, 0, 256), o=(192, 240, 1, 240, 0, 256), up=(192, 960, 1, 960, 0, 256),
        down=(192, 240, 1, 240, 0, 256))


@pytest.mark.parametrize("shape,want", M.MLP_SHAPES, ids=str)
def test_gpu_mlp_shapes_reach_their_plans(shape, want):
    dim, mlp, lens, text = shape
    got = M.projections([(n - text, text) for n in lens], dim, mlp)
    assert {k: got[k] for k in want} == want


@pytest.mark.parametrize("name", list(M.BLOCK_SHAPES) + list(M.SPLIT_K_SHAPES))
def test_gpu_block_shapes_reach_their_plans(name):
    shape, want = (M.BLOCK_SHAPES | M.SPLIT_K_SHAPES)[name]
    assert M.projections(M.segments(shape), shape.dim, shape.mlp_dim) == want


@pytest.mark.parametrize("name", list(M.FP8_SHAPES))
def test_gpu_fp8_shapes_reach_their_plans(name):
    shape, want = M.FP8_SHAPES[name]
    assert M.projections(M.segments(shape), shape.dim, shape.mlp_dim, fp8=True) == want


def test_chosen_plans_of_random_problems():
    """Whatever tile is chosen: a launch without the fixup has no cut tile, and the plan's schedule holds (every
    K step once, partial slots below 3 P)."""
    r = random.Random(1)
    checked = 0
    for _ in range(4000):
        batch, text = r.choice([1, 1, 2, 5]), r.choice([0, 1, 77, 512])
        most = r.randrange(4, 3000)  # image rows at most, per sample
        segs = [(r.randrange(0, most + 1), text) for _ in range(batch)]
        N, K, resid = 64 * r.randrange(1, 129), 64 * r.randrange(1, 257), r.random() < 0.5
        for tile, kstep in ((None, 64), (192, 128), (256, 128)):
            if kstep == 128 and K % 128:
                continue
            d = M.describe(segs, N, K, resid, tile, kstep)
            if d[0] == "small":
                continue
            if M.fixup_skipped(most, text, batch, N, K, tile or 192, kstep):
                assert d[2] == 1 and d[4] == 0, (segs, N, K, d)
            if checked < 300 and d[1] * (K // kstep) < 60000:
                check(d[1], M.WORKGROUPS, K // kstep)
                checked += 1


def test_schedule_random_cases():
    r = random.Random(0)
    for _ in range(600):
        T, P, nk = r.randint(0, 700), r.choice([1, 2, 7, 64, 255, 256]), r.randint(1, 200)
        check(T, P, nk)
        check(T, P, nk, cut_plan)
