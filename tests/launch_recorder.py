"""launches(): the kernels the library launches for given arguments, in order, found without a GPU (abi_c/launch_recorder.c)."""
import collections
import os
import re
import subprocess
import tempfile

from paper_2411_10958_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
Launch = collections.namedtuple("Launch", "kernel mangled grid block")
_BIN = None


def _recorder():
    global _BIN
    if _BIN is None:
        folder = tempfile.TemporaryDirectory()
        rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
        exe = os.path.join(folder.name, "launch_recorder")
        subprocess.run(["gcc", "-std=c11", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                        "-I", os.path.join(build.ROOT, "include"), "-o", exe, os.path.join(HERE, "abi_c", "launch_recorder.c"),
                        "-L", build.PKG, "-l:libsageattn.so", "-Wl,-rpath," + build.PKG, "-Wl,-rpath-link," + os.path.join(rocm, "lib")],
                       check=True)
        _BIN = exe, folder        # (the folder goes with the process)
    return _BIN[0]


def launches(calls):
    """calls: (entry point, fields of sage_attn_args) each.  Returns one (status, [Launch, ...]) per call."""
    text = "".join(" ".join([entry, *(f"{n}={int(x)}" for n, x in kw.items())]) + "\n" for entry, kw in calls)
    run = subprocess.run([_recorder()], input=text, capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stderr
    res, cur = [], []
    for line in run.stdout.splitlines():
        word = line.split()
        if word[0] == "status":
            res.append((int(word[1]), cur))
            cur = []
        else:
            cur.append(Launch(re.search(r"\d(k_[a-z0-9_]+?)(?:IL|E)", word[1])[1], word[1], tuple(map(int, word[2:5])), int(word[5])))
    assert len(res) == len(calls)
    return res
