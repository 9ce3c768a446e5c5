"""The persistent level driver's tickets and the server on them as a model of
CPU threads (tests/sanitize/ticket_protocol_model.cpp): under ThreadSanitizer,
with planted mistakes that it or a result has to show, and many times without
a sanitizer."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

SOURCE = os.path.join(ROOT, "tests", "sanitize", "ticket_protocol_model.cpp")


def run_model(tmp_path, plant, flags, reps):
    exe = str(tmp_path / "ticket_protocol_model")
    subprocess.check_call(["g++", "-std=c++17", "-pthread", f"-DPLANT={plant}", *flags, SOURCE, "-o", exe])
    return subprocess.run([exe, str(reps)], capture_output=True, text=True, timeout=300,
                          env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1 exitcode=66"))


TSAN = ["-O1", "-g", "-fsanitize=thread"]


def test_no_race_and_every_result_right(tmp_path):
    r = run_model(tmp_path, 0, TSAN, 20)
    assert "ThreadSanitizer" not in r.stderr, r.stderr[-4000:]
    assert r.returncode == 0 and r.stdout.strip() == "errors 0", r.stdout + r.stderr[-2000:]


def test_many_runs(tmp_path):
    r = run_model(tmp_path, 0, ["-O2"], 400)
    assert r.returncode == 0 and r.stdout.strip() == "errors 0", r.stdout[-3000:]


@pytest.mark.parametrize("plant,what", [
    (1, "a ticket written without release"),
    (2, "a finished tile counted without ordering"),
    (3, "a level's counters reset after the next ticket"),
    (4, "the level record written after its ticket"),
    (5, "the admission tail raised without release"),
    (6, "a completion record published without release"),
    (7, "a slot's constants kept for its next query"),
    (8, "a solo level's states written after the ticket"),
    (9, "level counts copied after the completion record"),
    (10, "the poll's ticket trusted instead of the add's"),
])
def test_planted_mistakes_show(tmp_path, plant, what):
    r = run_model(tmp_path, plant, TSAN, 20)
    assert "ThreadSanitizer: data race" in r.stderr or r.returncode != 0, f"not caught: {what}"
