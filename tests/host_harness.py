"""Compile a few lines of C++ against the library's headers that need no HIP
and run them: the host rules themselves, without a GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1501_00324_amd", "csrc")


def run_cpp(tmp_path, headers, body):
    """Words printed by `body` (the statements of main)."""
    src = tmp_path / "harness.cpp"
    src.write_text("#include <cstdio>\n#include <initializer_list>\n%s\nusing namespace fs;\nint main()\n{\n%s\n}\n" % (
        "\n".join('#include "%s"' % h for h in headers), body))
    exe = tmp_path / "harness"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()
