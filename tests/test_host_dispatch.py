"""The library's host code (which kernels a call takes, the control of a solve, what happens when
memory or a launch is refused) run on the CPU: the real sources linked with stand-ins for the HIP
runtime and the launchers (host_stubs.cpp), one scenario per process."""
import concurrent.futures
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_1811_00893_amd.csrc import build
    out = tmp_path_factory.mktemp("host")
    src = [os.path.join(build.HERE, s) for s in ("runtime.cpp", "solver.cpp", "capi.cpp", "dslash.hip")]
    src.append(os.path.join(ROOT, "tests", "host_stubs.cpp"))
    objs = [str(out / (os.path.basename(s) + ".o")) for s in src]

    def compile_one(pair):
        return subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-O1", "-fPIC", "-std=c++17", "-w", "-I", build.HERE, "-I",
                               os.path.join(ROOT, "include"), "-c", pair[0], "-o", pair[1]], capture_output=True, text=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(src)) as ex:
        for r in ex.map(compile_one, zip(src, objs)):
            assert r.returncode == 0, r.stderr[-4000:]
    exe = str(out / "host")
    nm = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True, check=True).stdout.split()
    none = sorted({f"-Wl,--defsym={n}=0" for n in nm if n.startswith("__hip_fatbin")})  # (no device code here)
    r = subprocess.run(["g++", "-o", exe] + objs + none + ["-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(program, scenario, **env):
    clean = {k: v for k, v in os.environ.items() if not k.startswith("WILSON_")}
    r = subprocess.run([program, scenario], env=dict(clean, **env), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_operator_keeps_the_order_of_the_tuned_hop(program):
    run(program, "operator_order")


def test_lost_one_launch_solve_goes_on_in_separate_launches(program):
    run(program, "one_launch_lost")
    run(program, "one_launch_off", WILSON_ONE_LAUNCH="0")


def test_one_launch_solves_share_the_room_of_the_device(program):
    run(program, "one_launch_room")


def test_a_load_makes_each_buffer_once(program):
    run(program, "load_allocates_once")


def test_a_shape_tuned_during_a_solve_does_not_fail_it(program):
    run(program, "shape_changes")


def test_timed_calls_run_the_hop(program):
    run(program, "timed_calls")


def test_plain_calls_give_back_what_they_keep(program):
    run(program, "plain_memory")
