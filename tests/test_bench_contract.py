"""Host-side parts of bench.py's contract: one GPU only, and the HBM traffic
figure read from the committed counter summary only while the kernel source
it was taken from is unchanged."""
import hashlib
import importlib.util
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench_contract_mod", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_more_than_one_gpu_is_refused():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert p.returncode != 0
    assert "one GPU" in p.stderr
    assert p.stdout.strip() == ""


def _traffic_block(name):
    text = open(os.path.join(ROOT, "profiles", name)).read()
    block = re.search(r"```traffic\n(.*?)```", text, re.S).group(1)
    return dict(line.split("=", 1) for line in block.strip().splitlines())


def test_traffic_follows_the_kernel_source_hash(tmp_path):
    b = _bench()
    name = "lm_head_8b_layer_p8192_traffic.md"
    kv = _traffic_block(name)
    files = kv["sources"].split()
    # the kernel and the headers that hold its helpers
    assert {os.path.basename(f) for f in files} >= {"gemm.hip", "gemm_common.hpp", "common.hpp"}
    src = [open(os.path.join(ROOT, f), "rb").read() for f in files]
    current = hashlib.sha256(b"".join(src)).hexdigest() == kv["sha256"]
    got = b.measured_traffic(name)
    if current:
        assert got == int(kv["bytes_per_launch"]) and got > 0
    else:
        assert got is None
    # a summary whose recorded hash does not match its sources gives null
    summary = open(os.path.join(ROOT, "profiles", name)).read()
    os.makedirs(tmp_path / "profiles")
    for f, data in zip(files, src):
        os.makedirs((tmp_path / f).parent, exist_ok=True)
        (tmp_path / f).write_bytes(data)
    b.ROOT = str(tmp_path)

    def traffic(sha):
        (tmp_path / "profiles" / name).write_text(summary.replace(kv["sha256"], sha))
        return b.measured_traffic(name)
    assert traffic("0" * 64) is None
    # and the untouched summary beside the same sources reads as before
    assert traffic(kv["sha256"]) == got
    # a change of any one of the files makes the figure stale
    now = hashlib.sha256(b"".join(src)).hexdigest()
    for f, data in zip(files, src):
        (tmp_path / f).write_bytes(data + b"\n")
        assert traffic(now) is None
        (tmp_path / f).write_bytes(data)
    assert traffic(now) == int(kv["bytes_per_launch"])
