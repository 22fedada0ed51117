"""The protocol of the packer of large tensors: every order in which its workgroups can run ends, however few of them run at
a time (CPU model that runs the kernel's own rules, see pack_ranges_model.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1905_10830_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("model") / "pack_ranges_model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "pack_ranges_model.cpp"), "-o", exe],
                   check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)


# one range for each workgroup, fewer ranges than workgroups, several rounds
@pytest.mark.parametrize("chunks,grid,images", [(4, 4, 1), (5, 4, 2), (2, 4, 1), (9, 3, 1), (8, 3, 1), (11, 3, 2), (6, 2, 1)])
@pytest.mark.parametrize("resident", [1, 2, 4])
def test_every_order_of_steps_ends(model, chunks, grid, images, resident):
    r = model("all", chunks, grid, images, resident)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("chunks,grid,images,resident", [(12544, 256, 64, 256), (12544, 256, 64, 7), (4097, 256, 32, 100), (138660, 256, 64, 200),
                                                         (30000, 256, 32, 1)])
def test_random_orders_of_a_whole_grid_end(model, chunks, grid, images, resident):
    r = model("walk", chunks, grid, images, resident, 2, 1)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("how", [("all", 9, 3, 1, 2), ("walk", 12544, 256, 64, 100, 2, 1)])
def test_the_model_sees_a_rule_that_gets_stuck(model, how):
    """Ranges by the workgroups' indices: one that runs may wait for one that has not started."""
    r = model(*how, "index")
    assert r.returncode == 2 and r.stdout.startswith("stuck"), r.stdout


def test_ranges_hold_every_chunk_once(model):
    r = model("cut")
    assert r.returncode == 0 and r.stdout.split() == ["ok", "18720"], r.stdout
