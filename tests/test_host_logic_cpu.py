"""Host and device logic that needs no device, compiled from the library's own headers with the host compiler."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_10872_amd", "csrc")


def run_host(tmp_path, name, *args):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-pthread", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe], check=True)
    done = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout.strip().endswith("ok"), done.stdout + done.stderr


def test_arrival_counters_return_to_zero(tmp_path):
    run_host(tmp_path, "arrivals")


def test_a_team_never_has_more_members_than_compute_units(tmp_path):
    run_host(tmp_path, "team_rows")


def test_teams_that_have_waited_are_admitted_in_the_order_of_their_requests(tmp_path):
    run_host(tmp_path, "admission")


def test_launches_of_a_team_are_short_and_shorter_where_others_wait(tmp_path):
    run_host(tmp_path, "launch_length")


def test_how_long_solves_keep_to_the_chain(tmp_path):
    run_host(tmp_path, "team_record")


def test_what_a_host_thread_throws_reaches_the_caller(tmp_path):
    run_host(tmp_path, "host_threads")
