"""Reuse of a context's batch tables (CPU): the product's knnf_api.cpp against the
fake HIP runtime of tests/fakehip, under AddressSanitizer and ThreadSanitizer.

A batched call takes the table that was used longest ago and has to wait for the
launch that used it, whatever has become of that launch's stream: destroyed while
the launch still ran, with another stream at its handle; the per-thread stream of
another thread, which has the caller's handle; a stream whose work a capture
recorded, to be replayed at any time.  And closing a server leaves its context, which
may be gone, alone; and a window's rows stay in range for every R.
"""
import os
import subprocess

import pytest

from test_server_fake import CSRC, FAKE, ROOT, oracle_obj  # noqa: F401

SOURCES = [os.path.join(CSRC, "knnf_api.cpp"), os.path.join(CSRC, "knnf_server.cpp"),
           os.path.join(FAKE, "fake_runtime.cpp"),
           os.path.join(FAKE, "fake_device.cpp"), os.path.join(FAKE, "test_batch_slots.cpp")]


@pytest.mark.parametrize("name,flags,env", [
    ("asan", ["-fsanitize=address,undefined"],
     {"ASAN_OPTIONS": "detect_leaks=1:abort_on_error=1", "UBSAN_OPTIONS": "halt_on_error=1"}),
    ("tsan", ["-fsanitize=thread", "-include", os.path.join(FAKE, "tsan_cond.h")],
     {"TSAN_OPTIONS": "halt_on_error=1"}),
], ids=["address", "thread"])
def test_tables_are_reused_after_their_launch(oracle_obj, name, flags, env):  # noqa: F811
    d, obj = oracle_obj
    exe = str(d / f"slots_{name}")
    cmd = (["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-ffp-contract=off", "-Wall",
            "-I", FAKE, "-I", os.path.join(ROOT, "include"), "-I", CSRC] + flags + SOURCES
           + [obj, "-lpthread", "-o", exe])
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0 and "sanitize" in r.stderr and "unrecognized" in r.stderr:
        pytest.skip(f"sanitizer not supported: {r.stderr[:200]}")
    assert r.returncode == 0, r.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, **env))
    assert run.returncode == 0, (run.stdout + run.stderr)[-4000:]
    assert run.stdout.split() == ["ok", "destroyed_stream", "ok", "per_thread_streams", "ok",
                                  "captured_batches", "ok", "server_closed_after_its_context", "ok",
                                  "whole_frame_windows"]
