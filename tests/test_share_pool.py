"""The pool of library-owned scratch buffers (csrc/share_pool.h) on a runtime of counters: who may get a buffer that
others have used, how many there are, what failures leave behind. Under the address and undefined-behaviour sanitizers."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_buffers_are_lent_in_order(tmp_path):
    exe = str(tmp_path / "share_pool_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=address,undefined",
                    os.path.join(HERE, "share_pool_driver.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr
