"""Item list of the walk form of the sweeps on the CPU: every value an item
waits for is published by an earlier one, every family's step and every
node's state is formed, and written, once."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("wpc") / "walk_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-pthread", os.path.join(ROOT, "tests", "native", "walk_plan_check.cpp"),
                    os.path.join(ROOT, "paper_2212_01110_amd", "csrc", "host_core.cpp"), "-o", exe], check=True)
    return exe


def _tree(children):
    """children(node, stage) per node of every stage but the last."""
    anc, prob, level, stage = [-1], [1.0], [0], 0
    while True:
        nxt = []
        for i in level:
            n = children(i, stage)
            for _ in range(n):
                anc.append(i)
                prob.append(prob[i] / n)
                nxt.append(len(anc) - 1)
        if not nxt:
            return anc, prob
        level, stage = nxt, stage + 1


def _uneven(seed, N):
    rng = np.random.default_rng(seed)
    return _tree(lambda i, t: 0 if t == N else int(rng.choice([1, 1, 2, 3])))


TREES = {"one": _tree(lambda i, t: 3 * (t < 1)), "chain": _tree(lambda i, t: 1 * (t < 70)),
         "binary": _tree(lambda i, t: 2 * (t < 9)), "split": _tree(lambda i, t: (2 if t < 4 else 1) * (t < 9)),
         "middle": _tree(lambda i, t: (1 if t in (0, 1, 4, 5) else 5) * (t < 6)), "uneven": _uneven(3, 7),
         "wide": _tree(lambda i, t: (40 if t == 1 else 1) * (t < 4))}


@pytest.mark.parametrize("name", list(TREES))
@pytest.mark.parametrize("nc", [1, 2, 8])
@pytest.mark.parametrize("max_chain,max_path,max_pieces", [(1, 0, 256), (1, 1, 256), (3, 2, 256), (100, 100, 256),
                                                           (100, 100, 7), (2, 100, 1)])
def test_items_cover_the_sweeps_in_order(driver, tmp_path, name, nc, max_chain, max_path, max_pieces):
    anc, prob = TREES[name]
    path = tmp_path / "case.txt"
    path.write_text(f"{len(anc)}\n{' '.join(map(str, anc))}\n{' '.join(map(repr, prob))}\n"
                    f"{nc} {max_chain} {max_path} {max_pieces}\n")
    res = subprocess.run([driver, str(path)], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.startswith("ok "), (res.stdout, res.stderr[-2000:])
