"""What the build runs, followed with a stand-in for the compiler."""
import os
import stat

from paper_2502_19811_amd import build

COMPILER = """#!/bin/sh
echo "$@" >> "$0.log"
while [ $# -gt 0 ]; do
  if [ "$1" = -o ]; then : > "$2"; fi
  shift
done
"""


def test_flags_reach_every_command_and_objects_lie_beside_the_output(tmp_path, monkeypatch):
    hipcc, out = str(tmp_path / "hipcc"), str(tmp_path / "out" / "lib.so")
    os.mkdir(os.path.dirname(out))
    with open(hipcc, "w") as f:
        f.write(COMPILER)
    os.chmod(hipcc, stat.S_IRWXU)
    monkeypatch.setenv("HIPCC", hipcc)
    before = sorted(os.listdir(build.PKG_DIR))
    assert build.build_library(extra_flags=["-DSOME_FLAG", "-Wl,--some-option"], out_path=out) == out
    with open(hipcc + ".log") as f:
        commands = f.read().splitlines()
    assert len(commands) == len(build.SOURCES) + 1
    for c in commands:
        assert "-DSOME_FLAG -Wl,--some-option" in c
        target = c.split(" -o ")[1].split()[0]
        assert target.startswith(os.path.dirname(out) + os.sep)
    assert os.listdir(os.path.dirname(out)) == ["lib.so"]      # the objects are gone
    assert sorted(os.listdir(build.PKG_DIR)) == before
