"""The served form on the CPU: the server's host code, its streams as threads,
and the persistent kernel with its parking and slot reuse."""
import os
import subprocess
import sys

import pytest

import emu_lib


@pytest.fixture(scope="module")
def library():
    return emu_lib.load_library()._name


@pytest.mark.parametrize("seed", range(1, 5))
def test_streams_of_jobs(library, seed):
    """Every job's result is the oracle's, and no stream stalls, with the
    streams on one to five hardware queues and arenas of different sizes."""
    r = subprocess.run([sys.executable, os.path.join(os.path.dirname(__file__), "server_stream.py"), library, str(seed), "3"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
