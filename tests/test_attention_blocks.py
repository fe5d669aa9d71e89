"""Block schedule of the bf16 prefill attention on the CPU: the header that the kernel runs, compiled into a host program that
walks it as the four waves do (tests/host_check/attention_blocks_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_waves_pass_the_same_tiles_and_take_every_key_once(tmp_path):
    exe = str(tmp_path / "attention_blocks_check")
    src = os.path.join(HERE, "host_check", "attention_blocks_check.cpp")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, src], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-3000:]
