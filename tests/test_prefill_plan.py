"""The cut of the column sweep into blocks and pieces, over shapes and over what a mask leaves of them (CPU, g++)."""
import importlib
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("plan") / "prefill_plan")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           os.path.join(HERE, "plan", "prefill_plan_main.cpp"), "-o", exe])

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
        assert r.returncode == 0, r.stdout[-3000:]
        return r.stdout
    return run


def test_no_empty_run_and_no_piece_beyond_the_workspace(plan):
    plan()


@pytest.mark.parametrize("module,want", [("test_gpu_prefill_rows", "rows, with normalisers rows"),
                                         ("test_gpu_prefill_one_chunk", "persistent wide 1 chunk, with normalisers persistent")])
def test_gpu_tests_reach_the_form_they_are_for(plan, module, want):
    for B, Mv, N, H, d, _, mask in importlib.import_module(module).SHAPES:
        assert plan(B, Mv, N, H, d, int(mask)).strip() == want, (B, Mv, N, H, d, mask)
