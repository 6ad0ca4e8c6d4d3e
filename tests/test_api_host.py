"""csrc/hack_api.cpp compiled for the host over a stand-in for the HIP runtime and the kernels (tests/host/): what the
entry points plan, upload and launch, without a GPU."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("api") / "api_check"
    src = os.path.join(ROOT, "tests", "host", "api_check.cpp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(ROCM, "include"), src, "-o", str(exe)], check=True)

    def run(name):
        r = subprocess.run([str(exe), name], capture_output=True, text=True)
        sys.stdout.write(r.stdout)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr[-2000:]
    return run


def test_tables_first_seen_during_a_capture_are_not_taken_for_uploaded(check):
    check("capture")


def test_steps_whose_outputs_lie_over_the_new_rows_move_them_first(check):
    check("out_over_new_rows")


def test_short_units_take_one_launch_and_every_unit_once(check):
    check("short_units")


def test_short_units_take_a_launch_of_their_own_where_that_spares_a_round(check):
    check("short_units_apart")


def test_a_step_table_holds_every_unit_once(check):
    check("step_tables")


def test_no_exception_crosses_the_abi_when_host_memory_runs_out(check):
    check("no_exceptions")


def test_float32_score_workspace_covers_every_launch_and_no_more(check):
    check("f32_workspace")


def test_remembered_steps_are_found_by_all_their_arguments(check):
    check("step_keys")


def test_attention_kernel_rule_and_its_override(check):
    check("attn_rule")


def test_a_step_and_single_attention_take_the_same_waves(check):
    check("split_waves")


def test_keys_in_halves_only_where_most_work_items_are_long(check):
    check("key_halves")


def test_short_compressing_steps_take_one_launch(check):
    check("whole_steps")


def test_score_item_sizes(check):
    check("score_items")
