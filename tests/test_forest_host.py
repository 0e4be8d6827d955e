"""CPU tests of the compiler's merge of a batch, built from its source with the address and undefined-behaviour
sanitizers: games deeper than 127 levels (the depth of a node once went through eight bits), alone in the batch
and beside shallow ones."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def forest(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("native") / "forest")
    csrc = os.path.join(ROOT, "paper_2609_11923_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", csrc,
                    os.path.join(HERE, "native", "forest.cpp"), os.path.join(csrc, "compiler.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("depths", [(1, 2), (3, 1, 5), (127, 126), (128, 2), (3, 200, 129), (300, 300, 300)])
def test_batches_of_deep_games(forest, depths):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([forest, *map(str, depths)], capture_output=True, text=True, env=env, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr[:2000]
