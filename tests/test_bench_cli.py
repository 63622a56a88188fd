"""bench.py's command line, as far as it can be checked without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], capture_output=True, text=True,
                          timeout=120)


def test_more_than_one_gpu_is_refused_with_a_message():
    r = _run("--gpus", "2")
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr


def test_a_distributed_launch_is_refused_too():
    env = dict(os.environ, WORLD_SIZE="2")
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py")], capture_output=True, text=True, timeout=120,
                       env=env)
    assert r.returncode != 0 and "ONE GPU" in r.stderr


def test_defaults_measure_the_steady_state():
    r = _run("--help")
    assert r.returncode == 0
    for flag in ("--steps", "--warmup", "--workload", "--no-cpu-baseline", "--no-next-rows", "--option"):
        assert flag in r.stdout


def test_graft_entry_has_build_and_smoke():
    sys.path.insert(0, ROOT)
    import __graft_entry__ as g
    assert callable(g.build) and callable(g.smoke)


def test_refresh_is_priced_on_the_pipe_that_does_it():
    """Short bases or few gradients stay on the fp64 matrix pipe, whatever the slice length."""
    sys.path.insert(0, ROOT)
    import bench
    from paper_1811_03617_amd import WORKLOADS
    for name, L, want in (("vgg16", 32, True), ("vgg16", 1, True), ("vgg16_bf16", 32, True), ("vgg16_bf16", 2, False),
                          ("alexnet", 16, False), ("tiny", 8, False)):
        assert bench.fit_on_int8_pipe(WORKLOADS[name], L) == want
