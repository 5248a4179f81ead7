"""Launches that would leave much of the chip idle run on smaller tiles than
their class's.  Host: the lists they run on cover every output exactly once.
GPU: an element's value does not depend on the tile that computed it, nor on
what it was launched with -- a
matrix on its own (small tiles) and the same matrix among enough others to
fill the chip (256 tiles with their half tiles and edge strips, or the class
tile) give bitwise the same W, M and O."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2606_27153_amd.optim import MuonPlan
from paper_2606_27153_amd.workloads import WORKLOAD_KEYS, custom_workload, get_workload, make_grads, make_state

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lists_check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("exec") / "exec_lists_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "exec_lists_check.cpp"),
                    os.path.join(ROOT, "paper_2606_27153_amd", "csrc", "plan.cpp"), "-o", str(exe)], check=True)
    return str(exe)


def _run(exe, shapes, precision):
    out = subprocess.run([exe, str(precision)], input="\n".join(f"{r} {c}" for r, c in shapes), capture_output=True,
                         text=True)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr
    return [int(v) for v in out.stdout.split()[1:]]


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_lists_cover_outputs(lists_check, precision):
    rng = np.random.default_rng(7)
    used = np.zeros(7, int)
    for n in (1, 2, 3, 5, 9, 17):
        for _ in range(6):
            shapes = [(int(rng.integers(1, 2600)), int(rng.integers(1, 2600))) for _ in range(n)]
            used += _run(lists_check, shapes, precision)
    for r, c in ((1, 1), (64, 64), (65, 65), (256, 256), (257, 257), (384, 385), (2048, 5632), (4096, 14336)):
        used += _run(lists_check, [(r, c)], precision)
    # every kernel the precision has is chosen somewhere
    assert used[1] and used[3] and (precision == 1 or (used[0] and used[2])), used
    # the tiny set's two groups advance together, the 8B set's do not
    if precision == 0:
        ragged = [(65, 200), (200, 65), (130, 700), (700, 130), (257, 513), (513, 257), (1000, 1000), (96, 4304),
                  (7, 13), (1152, 1200), (300, 300)]
        assert _run(lists_check, ragged, 0)[4:] == [0, 1, 0]   # its side groups share launches
        tiny, big = (_run(lists_check, [(m.rows, m.cols) for m in get_workload(k).matrices], 0) for k in ("tiny", "8b"))
        assert tiny[4:] == [0, 0, 1] and big[5:] == [0, 0]
    for key in WORKLOAD_KEYS:
        _run(lists_check, [(m.rows, m.cols) for m in get_workload(key).matrices], precision)


# one matrix shape, and how many of it leave the small tiles: one-tile and
# two-tile squares, half tiles and edge strips on both sides, a tall and a wide
# Gram-space matrix, odd columns, the 128 and 64 classes; one-tile matrices whose
# square products of either form run on the 256 tile, with a wave block of
# padding and without
SHAPES = [((180, 700), 600), ((256, 400), 1100), ((256, 256), 300), ((512, 512), 150), ((640, 640), 120),
          ((384, 1100), 150), ((1152, 385), 150),
          ((300, 301), 200), ((130, 700), 300), ((96, 520), 400), ((40, 200), 900)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["bf16", "fp16", "fp32"])
@pytest.mark.parametrize("shape,many", SHAPES, ids=[f"{s[0]}x{s[1]}" for s, _ in SHAPES])
def test_value_does_not_depend_on_the_tile(shape, many, precision):
    dev = "cuda:0"
    got = []
    for n in (1, many):
        wl = custom_workload([shape] * n, seed=71)
        plan = MuonPlan([(m.rows, m.cols, m.param, m.grad) for m in wl.matrices], precision=precision)
        params, moms = make_state(torch, wl, dev)
        grads = make_grads(torch, wl, 0, dev)
        outs = [torch.full(shape, float("nan"), device=dev)] + [None] * (n - 1)
        plan.step(params, grads, moms, lr=0.02, momentum=0.95, weight_decay=0.01, ns_steps=5, update_out=outs)
        torch.cuda.synchronize()
        got.append((params[0], moms[0], outs[0]))
        plan.close()
    for a, b in zip(*got):
        assert torch.isfinite(a).all()
        assert torch.equal(a, b)


# waves of small groups of every kind (Eq. 2 and Gram space on the 256, 128 and
# 64 classes, fp32 for small m under bf16; odd columns, tall matrices): all
# merged, side groups sharing launches beside a main group, side groups on
# streams of their own beside a large one
SMALL = [(256, 768), (768, 256), (300, 301), (130, 700), (96, 520), (70, 72), (40, 200), (200, 33), (64, 64), (512, 512)]
WAVES = {"merged": SMALL,
         "sides merged": [(257, 513), (513, 257), (130, 700), (96, 4304), (1000, 1000), (7, 13), (1152, 1200), (300, 300),
                          (65, 200)],
         "side streams": SMALL + [(1024, 1024)] * 40}


def test_wave_modes(lists_check):
    assert [_run(lists_check, WAVES[k], 0)[4:] for k in WAVES] == [[0, 0, 1], [0, 1, 0], [1, 0, 0]]


# groups with a launch of more than 1024 class tiles: (shapes with counts,
# precision); left out of their chains' estimates, such launches made a merged
# wave look faster (measured apart / merged: 231 / 257, 221 / 236, 866 / 946 us)
FILLING = [([(70, 512, 102), (24, 512, 77), (200, 256, 31), (24, 700, 40)], 2),
           ([(32, 1500, 51), (200, 700, 9), (384, 256, 36)], 2),
           ([(200, 256, 57), (32, 512, 28), (56, 1000, 44), (70, 700, 43), (16, 1000, 39), (24, 512, 48),
             (256, 1500, 15)], 1)]


@pytest.mark.parametrize("shapes,precision", FILLING)
def test_groups_that_fill_the_chip_are_not_merged(lists_check, shapes, precision):
    assert _run(lists_check, [(r, c) for r, c, n in shapes for _ in range(n)], precision)[4:] == [1, 0, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["bf16", "fp16"])
@pytest.mark.parametrize("wave", list(WAVES))
def test_groups_run_together_match_each_matrix_alone(wave, precision):
    # several steps, one matrix with a zero gradient, one without a gradient:
    # bitwise each matrix on its own; then the same step captured in a graph and
    # replayed between eager steps
    dev = "cuda:0"
    wl = custom_workload(WAVES[wave], seed=73)
    kw = dict(lr=0.02, momentum=0.95, weight_decay=0.01, ns_steps=5)
    descs = [(m.rows, m.cols, m.param, m.grad) for m in wl.matrices]
    plan = MuonPlan(descs, precision=precision)
    params, moms = make_state(torch, wl, dev)
    alone = [(p.clone(), m.clone()) for p, m in zip(params, moms)]
    plans = [MuonPlan([d], precision=precision) for d in descs[:10]]

    def check(grads, what):
        for i, q in enumerate(plans):
            q.step([alone[i][0]], [grads[i]], [alone[i][1]], **kw)
        torch.cuda.synchronize()
        for i in range(len(plans)):
            assert torch.equal(params[i], alone[i][0]) and torch.equal(moms[i], alone[i][1]), (descs[i], what)

    for step in range(2):
        grads = make_grads(torch, wl, step, dev)
        grads[2].zero_()
        grads[3] = None if step else grads[3]
        plan.step(params, grads, moms, **kw)
        check(grads, f"step {step}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.step(params, grads, moms, **kw)
    for replay in range(4):
        for g, new in zip(grads, make_grads(torch, wl, 2 + replay, dev)):
            if g is not None:
                g.copy_(new)
        if replay == 2:
            plan.step(params, grads, moms, **kw)
            check(grads, "eager between replays")
        graph.replay()
        check(grads, f"replay {replay}")
    for q in plans + [plan]:
        q.close()


# enough matrices with a half tile (m padded to 128 past a multiple of 256) that
# the square products of both forms stay on the 256 tile
HALF_SET = [(1152, 1700)] * 36 + [(1700, 1152)] * 36 + [(640, 640)] * 180


@pytest.mark.parametrize("precision", [0, 2])
def test_half_tile_set_stays_on_the_256_tile(lists_check, precision):
    # three kinds of launch for each of the two groups, no small-tile list
    assert _run(lists_check, HALF_SET, precision)[:4] == [6, 0, 0, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["bf16", "fp16"])
def test_half_tiles_match_the_oracle(precision):
    from parity_utils import assert_parity, run_parity
    wl = custom_workload(HALF_SET, seed=74)
    plan = MuonPlan([(m.rows, m.cols, m.param, m.grad) for m in wl.matrices], precision=precision)
    assert [plan.matrix_info(i)["m_pad"] for i in (0, 71, 72)] == [1152, 1152, 640]
    res = run_parity(wl, precision=precision, steps=1, plan=plan, check=[0, 71, 72, 251])
    plan.close()
    assert_parity(res, precision, "half tiles on the 256 tile")
