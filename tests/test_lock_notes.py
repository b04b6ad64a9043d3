"""The notes that waiters of the per-file miss lock leave for its holder, as a CPU thread model under
ThreadSanitizer on the device's encodings (tests/csrc/lock_notes_model.cpp says what it checks):
files that share a row of notes, files opened again, launches of different largest windows; and
planted mistakes that the checks must catch."""
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
    out = str(tmp_path_factory.mktemp("lnm") / "lock_notes_model")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread",
                           "-I", os.path.join(ROOT, "include"), "-o", out,
                           os.path.join(ROOT, "tests", "csrc", "lock_notes_model.cpp")])
    return out


def _run(model, args, deadline_s=60):
    env = dict(os.environ, TSAN_OPTIONS="halt_on_error=1 exitcode=66", LNM_DEADLINE_S=str(deadline_s))
    return subprocess.run([model] + [str(a) for a in args], capture_output=True, text=True, timeout=200, env=env)


@pytest.mark.parametrize("files,threads,misses", [(1, 24, 80), (2, 24, 160), (3, 48, 120), (16, 32, 400)])
def test_every_waiter_is_decided_for_on_its_own_miss(model, files, threads, misses):
    for seed in (1, 2):
        r = _run(model, ["notes", files, threads, misses, seed])
        assert r.returncode == 0 and r.stdout.strip().endswith("-> ok"), r.stdout + r.stderr[-3000:]
        assert int(r.stdout.split(": ")[1].split()[0]) > 0, r.stdout


@pytest.mark.parametrize("mode,files,what", [("no-tag", 2, "another miss"), ("note-first", 1, "another miss"),
                                             ("pass-over", 2, "deadline")])
def test_a_planted_mistake_is_caught(model, mode, files, what):
    r = _run(model, [mode, files, 24, 80 * files, 1], deadline_s=10)
    assert r.returncode == 1 and what in r.stderr, r.stdout + r.stderr[-3000:]
