"""The per-file miss lock as a CPU thread model, under ThreadSanitizer (tests/csrc/miss_lock_model.cpp
says what it checks): holders that decide for the waiters behind them, holders that decide for
themselves alone, many threads and few, few pages (windows meet) and many; and a planted mistake,
a waiter whose outcome the holder forgets, which the deadline must catch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    out = str(tmp_path_factory.mktemp("mlm") / "miss_lock_model")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread",
                           "-I", os.path.join(ROOT, "include"), "-o", out,
                           os.path.join(ROOT, "tests", "csrc", "miss_lock_model.cpp")])
    return out


def _run(model, args, deadline_s=60):
    env = dict(os.environ, TSAN_OPTIONS="halt_on_error=1 exitcode=66", MLM_DEADLINE_S=str(deadline_s))
    return subprocess.run([model] + [str(a) for a in args], capture_output=True, text=True, timeout=200, env=env)


@pytest.mark.parametrize("mode,threads,misses,pages", [
    ("batch", 2, 2000, 256), ("batch", 24, 800, 64), ("batch", 24, 800, 2048), ("batch", 80, 300, 512),
    ("single", 24, 400, 512)])
def test_lock_protocol(model, mode, threads, misses, pages):
    for seed in (1, 2):
        r = _run(model, [mode, threads, misses, pages, seed])
        assert r.returncode == 0 and r.stdout.strip().endswith("-> ok"), r.stdout + r.stderr[-3000:]


def test_a_forgotten_outcome_is_caught(model):
    r = _run(model, ["drop-taken", 24, 400, 512, 1], deadline_s=5)
    assert r.returncode == 1 and "deadline" in r.stderr, r.stdout + r.stderr[-3000:]
