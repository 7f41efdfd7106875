"""Every pair of layouts that an apply of residual ranks above 2 can run in: the shrink
by k_shrink (row) or k_shrink_wide (wide), the expand in the row or the quad layout,
at sizes where the rule of salt_launch.h chooses it (checked with the same code,
built for the host), with ranks at the edges of the 8-rank passes, the 16-rank
chunks and the row groups, tiles that hold narrow and wide ranks side by side,
tokens with and without a centroid, rows past a step or a chunk by eight elements.
Integer inputs, bit-exact, on the GPU, and with smaller tables (and the rule's
sizes with them) on the CPU build of the kernel sources under AddressSanitizer."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2608_03579_amd import synth
from tests import cpu_build
from tests.test_gpu_tiles import _run_all
from tests.test_host_kernels import _check
from tests.test_launch_walk import CSRC, HERE

SHAPES = [("a", 264, 2056), ("b", 2056, 264), ("c", 648, 1032)]
DEEP = [("a", 4104, 72), ("b", 72, 8)]
LONG = [("a", 24584, 72)]

CASES = [
    # name, dtype, shapes, C, r_c, T, slots, ranks of users with a centroid, ranks of users without, M, shrink, expand
    ("decode ranks 3-6", "bf16", SHAPES, 5, 24, 60, 40, (3, 5, 6), (0, 1), 16, "row", "quad"),
    ("ranks 0-8", "bf16", SHAPES, 2, 40, 150, 30, (0, 1, 7, 8), (8,), 32, "row", "row"),
    ("ranks 9-12", "bf16", SHAPES, 1, 72, 200, 60, (9, 11, 12), (), 64, "row", "quad"),
    ("ranks 9-12, shared rows", "bf16", SHAPES, 1, 72, 210, 12, (9, 12), (), 64, "wide", "quad"),
    ("ranks 7-8, distinct users", "bf16", SHAPES, 8, 24, 310, 300, (7, 8), (), 32, "row", "quad"),
    ("ranks 9-12, long groups", "bf16", SHAPES, 1, 16, 420, 20, (1, 9, 12), (), 128, "row", "quad"),
    ("ranks 8-16, long groups", "bf16", SHAPES, 1, 64, 420, 20, (8, 15, 16), (), 128, "row", "row"),
    ("ranks 3-5, long groups", "bf16", SHAPES, 1, 56, 400, 20, (3, 4, 5), (), 128, "row", "quad"),
    ("no centroids, few users", "bf16", SHAPES, 0, 0, 150, 10, (), (1, 9, 16), 64, "row", "row"),
    ("no centroids, ranks 4-8", "bf16", SHAPES, 0, 0, 70, 30, (), (4, 8), 32, "row", "quad"),
    ("tail, distinct users", "bf16", SHAPES, 8, 32, 340, 150, (0, 1, 3, 8, 9), (15, 16, 17, 33, 34), 32, "wide", "quad"),
    ("tail, few users", "bf16", SHAPES, 4, 16, 210, 12, (1, 2), (16, 17, 18), 32, "wide", "row"),
    ("tail, short groups", "bf16", SHAPES, 25, 64, 340, 150, (1, 2, 8), (65, 66, 72), 16, "row", "quad"),
    ("tail, little work", "bf16", SHAPES, 3, 24, 48, 12, (1, 2), (25, 26), 16, "row", "row"),
    ("tail, long groups", "bf16", SHAPES, 2, 48, 1300, 60, (1, 2, 7), (49, 50), 128, "wide", "quad"),
    ("rank 24, long groups", "bf16", SHAPES, 2, 32, 1300, 20, (17, 23, 24), (), 128, "wide", "row"),
    ("rank 32, distinct users", "bf16", SHAPES, 4, 40, 380, 200, (31, 32), (), 32, "row", "quad"),
    ("tail, r_c 128", "bf16", SHAPES, 6, 128, 300, 40, (1, 2), (40, 72), 32, "row", "row"),
    ("few 64-token tiles", "bf16", DEEP, 8, 16, 3000, 64, (3, 16), (), 64, "wide", "row"),
    ("rows are the traffic", "bf16", LONG, 0, 0, 512, 140, (), (15, 16), 64, "wide", "row"),
    ("fp32, no centroids", "f32", SHAPES, 0, 0, 180, 40, (), (1, 5, 16), 16, "wide", "quad"),
    ("fp32, no centroids, little work", "f32", SHAPES, 0, 0, 60, 20, (), (3, 8), 16, "row", "quad"),
    ("fp32, centroids", "f32", SHAPES, 2, 24, 70, 20, (1, 5, 20), (), 16, "row", "row"),
    ("fp32, centroids, rank 4", "f32", SHAPES, 3, 8, 600, 200, (3, 4), (), 16, "row", "quad"),
]
IDS = [c[0] for c in CASES]
SMALL = [("a", 72, 136), ("b", 264, 24), ("c", 8, 264)]


def _workload(name, dtype, shapes, C, r_c, T, n_slots, with_c, without, *_):
    """Users with a centroid and users without (a fifth of them where there are both), every rank of each list
    occurring; tokens over all users, and for long groups over one centroid alone."""
    rng = np.random.default_rng([2608, 3579, 92, len(name), T])
    n_without = n_slots if not with_c else (0 if not without else max(len(without), n_slots // 5))
    slot_rank = np.concatenate([np.resize(np.asarray(without, np.int32), n_without),
                                np.resize(np.asarray(with_c, np.int32), n_slots - n_without)]).astype(np.int32)
    user_c = np.concatenate([np.full(n_without, -1), np.arange(n_slots - n_without) % max(C, 1)]).astype(np.int32)
    order = rng.permutation(n_slots)
    slot_rank, user_c = slot_rank[order], user_c[order]
    tok_u = np.concatenate([np.arange(n_slots), np.arange(T - n_slots) % n_slots]).astype(np.int32)
    rng.shuffle(tok_u)
    return synth.Workload(cfg=9, seed=len(name) + T, name="layouts", dtype=dtype, tables=shapes, n_centroids=C, r_c=r_c,
                          n_slots=n_slots, r_u_max=int(slot_rank.max()), slot_rank=slot_rank, tok_c=user_c[tok_u],
                          tok_u=tok_u, gamma=None, y0_kind="int", exact=True)


@pytest.fixture(scope="module")
def layouts(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("layouts") / "layouts")
    subprocess.run(["g++", "-std=c++17", "-O1", "-DSALT_HOST_ONLY", f"-I{CSRC}",
                    os.path.join(HERE, "host_checks", "layouts.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def _chosen(exe, w):
    slots = np.unique(w.tok_u)
    args = [4 if w.dtype == "f32" else 2, w.T, w.n_centroids, w.r_c, len(slots), int(w.slot_rank[slots].sum()),
            len(w.tables)]
    for _, i, o in w.tables:
        args += [i, o]
    for c in range(-1, w.n_centroids):
        of = w.tok_u[w.tok_c == c]
        args += [len(of), int(w.slot_rank[of].max(initial=0))]
    out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout.split()
    return int(out[0]), ("row", "wide")[int(out[1])], ("row", "quad")[int(out[2])]


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_the_rule(case, layouts):
    assert _chosen(layouts, _workload(*case)) == case[-3:]


@pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")
@pytest.mark.parametrize("case", [c for c in CASES if c[5] <= 210], ids=[c[0] for c in CASES if c[5] <= 210])
def test_on_the_cpu(case, tmp_path):
    _check(_workload(*case[:2], SMALL, *case[3:]), tmp_path, case[-3], exact=True)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_on_the_gpu(case):
    print(f"\n[gpu case] layouts: {case[0]}", flush=True)
    _run_all(_workload(*case), want_m=case[-3], exact=True)
