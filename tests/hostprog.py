"""Host programs over the library's internal header, for what its inline functions compute (nothing runs
on a GPU)."""
import subprocess

from paper_2510_09997_amd import build


def run(tmp_path, body):
    """Compiles main(){ body } for the host and returns what it prints."""
    src, exe = tmp_path / "host.hip", tmp_path / "host"
    src.write_text('#include <stdio.h>\n#include "clod_internal.h"\nusing namespace clod;\nint main() {\n'
                   + body + "\nreturn 0;\n}\n")
    cmd = [build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-I", build.CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, cwd=tmp_path)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-3000:])
    return r.stdout
