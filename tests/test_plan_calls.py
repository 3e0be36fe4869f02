"""What calls are planned as, where only a handle's state shows it: the table
of selections under several threads, and limits on the workspace.  The library's host code is compiled
alone and run on the CPU."""
import os
import subprocess

import pytest

from paper_2609_16389_amd import build

_SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "plan_calls.cpp")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "plan_calls")
    # (the symbol of the GPU code stays unresolved: nothing here launches)
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-pthread",
                    "-I" + os.path.join(build.ROOT, "include"), _SRC, "-Wl,--unresolved-symbols=ignore-all", "-o", exe],
                   check=True)

    def run(*args):
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, "%s: status %d\n%s%s" % (args, r.returncode, r.stdout, r.stderr)
        return r.stdout
    return run


@pytest.mark.parametrize("count", [1, 2, 4])
def test_threads_share_a_table(host, count):
    """Python threads share one handle per stream, and the interpreter's lock
    is not held during a call."""
    host("threads", count)


def test_both_plans_of_a_shape_are_kept(host):
    """With and without the persistent kernel: neither lookup evicts the other."""
    host("kept")


def test_limits_on_the_workspace(host):
    """xgemm_run_noalloc takes a call exactly if xgemm_run's plan fits the
    static array, and then runs that plan; no limit refuses or changes a call
    whose plan keeps it."""
    host("limits")


def test_batched_plans(host):
    """The same of batched calls; and a launch whose kernel does not apply
    leaves the selected tile plan as it was."""
    host("batches")


def test_batched_parity_cases_run_what_they_name(host):
    """The kernels that the batched parity tests say they reach."""
    from test_direct_kernel import BATCHES
    from test_gpu_parity import BATCH_ROUTES
    for case, route in {**BATCH_ROUTES, **{s + (0, False): "direct" for s in BATCHES}}.items():
        assert host("batch_route", *(int(v) for v in case)).strip() == route, case


def test_streaming_loads_of_b(host):
    """By B's size and only over rows that are whole cache lines."""
    host("streams")


def test_k_splits_of_decoding_steps(host):
    """No K split that runs two workgroups on a few CUs and one on the others."""
    host("doubled_up")


def test_k_splits_with_odd_rows(host):
    """64 x 64 blocks are charged what odd rows of A cost them in a K split."""
    host("odd_rows")
