"""Read-outs of a handle whose device is not the current one, or whose stream is under capture: the
library's objects linked against a stand-in HIP runtime with two devices (tests/host_read_out_main.cpp),
which needs no GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_read_out_on_the_handles_device(tmp_path):
    from paper_1307_3711_amd import build as B
    objs = [os.path.join(B.HERE, "_build", os.path.splitext(s)[0] + ".o") for s in B.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        pytest.skip("the library's objects are not built")
    main_o, exe = str(tmp_path / "main.o"), str(tmp_path / "read_out")
    flags = [f for f in B.FLAGS if f != "-shared"]
    subprocess.check_call(["hipcc"] + flags + ["-x", "hip", "-c", "-o", main_o,
                                               os.path.join(HERE, "host_read_out_main.cpp")], stderr=subprocess.DEVNULL)
    # the C++ linker alone: every HIP symbol is the stand-in's
    subprocess.check_call(["g++", "-o", exe, main_o] + objs)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "bad 0" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
