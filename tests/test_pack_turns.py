"""The protocol inside the packer of large tensors: every order in which its wavefronts can run ends (CPU model that runs the
kernel's own rules, see pack_turns_model.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1905_10830_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("model") / "pack_turns_model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "pack_turns_model.cpp"), "-o", exe],
                   check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)


@pytest.mark.parametrize("waves,images,turns", [(1, 2, 20), (2, 2, 20), (2, 3, 8), (2, 4, 8), (3, 2, 3), (3, 3, 2)])
def test_every_order_of_steps_ends(model, waves, images, turns):
    r = model("all", waves, images, turns)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("images", [2, 3, 4])
def test_random_orders_of_fifteen_packers_end(model, images):
    for turns, runs in ((2, 1500), (5, 600), (40, 60)):
        r = model("walk", 15, images, turns, runs, images)
        assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("waves,images", [(3, 2), (15, 2), (15, 3), (15, 4)])
def test_the_model_sees_a_rule_that_gets_stuck(model, waves, images):
    """Chunks dealt without a limit: a packer may wait for the place of a turn whose last chunk it has in hand."""
    r = model("all", 3, 2, 3, "counter") if waves == 3 else model("walk", waves, images, 8, 2000, 1, "counter")
    assert r.returncode == 2 and r.stdout.startswith("stuck"), r.stdout
