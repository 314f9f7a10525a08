"""Builds a small host program around the library's own headers and runs it."""
import subprocess

from paper_2401_09721_amd import build


def run(tmp_path, head, body, *args):
    """Compile `head` and `body` for the host (no device code) and return the
    words that the program prints."""
    src, obj, exe = tmp_path / "t.hip", tmp_path / "t.o", tmp_path / "t"
    src.write_text("#include <cstdio>\n#include <cstdlib>\n" + head + "using namespace fgbd;\n" + body)
    subprocess.run([build.hipcc(), "--offload-host-only", "-std=c++17", "-O1", f"-I{build.INCLUDE}", f"-I{build.CSRC}",
                    "-c", str(src), "-o", str(obj)], check=True, capture_output=True, timeout=110)
    subprocess.run([build.hipcc(), str(obj), "-o", str(exe)], check=True, capture_output=True, timeout=110)
    out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True, timeout=30)
    return out.stdout.split()
