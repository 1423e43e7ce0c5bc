"""How far the decoders' stream readers read, under AddressSanitizer and UndefinedBehaviorSanitizer on the CPU:
tests/sanitize/streams.cc compiles them from huff_decode.cuh and tree_walk.cuh (tests/sanitize/shim stands in for HIP's
headers) and runs them over records that are followed by the slack they are promised and by nothing else."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parent.parent
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-g", "-O1"]


@pytest.mark.skipif(shutil.which("gcc") is None or shutil.which("g++") is None, reason="needs gcc and g++")
def test_stream_readers_stay_inside_a_record_and_its_slack(tmp_path):
    obj, exe = tmp_path / "oracle.o", tmp_path / "streams"
    subprocess.run(["gcc", "-std=c99", *SAN, "-ffp-contract=off", "-c", str(ROOT / "oracle" / "kvcomp_oracle.c"), "-o", str(obj)],
                   check=True)
    subprocess.run(["g++", "-std=c++17", *SAN, "-Wall", "-Wno-attributes", "-Wno-unknown-pragmas",
                    "-I", str(ROOT / "tests" / "sanitize" / "shim"), str(ROOT / "tests" / "sanitize" / "streams.cc"), str(obj),
                    "-o", str(exe), "-lm"], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600,
                       env={"ASAN_OPTIONS": "detect_leaks=1:verify_asan_link_order=0", "UBSAN_OPTIONS": "print_stacktrace=1"})
    assert r.returncode == 0, r.stdout[-4000:]
    assert "streams driver: ok" in r.stdout
