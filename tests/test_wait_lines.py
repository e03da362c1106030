"""Pinned result words of waited extracts (tests/c/wait_lines.cpp, on the host
with a counting allocator)."""
import os
import subprocess
import threading

import pytest
import torch

from paper_0912_0947_amd import api, inputs
from paper_0912_0947_amd._lib import E_BUFFER, LsbError

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lines_are_taken_and_given_back(tmp_path):
    exe = str(tmp_path / "wait_lines")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-pthread",
                           os.path.join(HERE, "c", "wait_lines.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr


@pytest.mark.gpu
def test_waited_extracts_from_threads_that_come_and_go():
    """Three rounds of new threads, each with its own stream, message length
    and messages: every waited extract returns its own length and bytes, and
    calls that fail in between (header, buffer) leave the others alone."""
    from gpu_helpers import DEV

    failures = []

    def worker(t):
        try:
            stream = torch.cuda.Stream()  # default priority
            with torch.cuda.stream(stream):
                cover = torch.from_numpy(inputs.random_bytes(40000 + 16 * t, 4611, t)).to(DEV)
                for rep in range(20):
                    msg = torch.from_numpy(inputs.random_bytes(1000 + 37 * t + rep, 4612, t, rep)).to(DEV)
                    stego = api.embed(cover, msg, 1 + t % 8)
                    assert torch.equal(api.extract_sync(stego, 1 + t % 8), msg), (t, rep)
                    with pytest.raises(LsbError) as e:
                        api.extract_sync(stego, 1 + t % 8, out=torch.empty(7, dtype=torch.uint8, device=DEV))
                    assert e.value.code == E_BUFFER
        except BaseException as e:  # noqa: B036 (reported by the test's own thread)
            failures.append((t, e))

    for first in (0, 6, 12):
        threads = [threading.Thread(target=worker, args=(t,)) for t in range(first, first + 6)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert not failures, failures
