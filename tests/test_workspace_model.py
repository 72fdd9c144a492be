"""The kept temporaries on the CPU, against a model of the HIP calls with
vector clocks (tests/workspace_model): no block is handed out or given back
while work that may still be running uses it, whatever streams are destroyed
and take each other's addresses."""

import os
import subprocess

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "workspace_model")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("workspace") / "model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-I", HERE,
                    os.path.join(HERE, "model.cpp"), "-o", exe], check=True)

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (args, r.stdout, r.stderr)
        return r.stdout
    return run


@pytest.mark.parametrize("scenario", ["address", "address_unscoped"])
def test_a_new_stream_at_an_old_address(model, scenario):
    model(scenario)


def test_partial_rows_go_with_their_graph(model):
    model("graphs")


def test_idle_memory_is_given_back_for_an_allocation(model):
    model("memory")


def test_idle_memory_has_a_limit(model):
    model("limits")


def test_random_calls(model):
    for seed in range(50):
        model("random", seed)


def test_host_memory_that_runs_out(model):
    """No exception leaves the library, and no order is lost."""
    for seed in range(30):
        model("host_memory", seed)
