"""The build makes both libraries at once and says why it fails (the compiler is a stand-in here; no GPU, nothing is compiled)."""
import os

import pytest

from paper_2501_15021_amd import build as akvq_build


@pytest.fixture
def stand_in(tmp_path, monkeypatch):
    """A compiler that notes its arguments, writes what it is asked for and fails where FAIL is among them."""
    def install(fail):
        path, log = tmp_path / "hipcc", tmp_path / "log"
        path.write_text(f"""#!/bin/sh
echo "$@" >> {log}
case "$*" in *{fail}*) echo "what went wrong" >&2; exit 1;; esac
while [ $# -gt 0 ]; do if [ "$1" = -o ]; then echo new > "$2"; fi; shift; done
""")
        path.chmod(0o755)
        csrc, lib, nowait = tmp_path / "csrc", tmp_path / "libakvq.so", tmp_path / "libakvq_nowait.so"
        csrc.mkdir()
        for old in (lib, nowait):
            old.write_text("old")
        monkeypatch.setattr(akvq_build, "HIPCC", str(path))
        monkeypatch.setattr(akvq_build, "CSRC", str(csrc))
        monkeypatch.setattr(akvq_build, "LIB", str(lib))
        monkeypatch.setattr(akvq_build, "NOWAIT", str(nowait), raising=False)
        monkeypatch.setattr(akvq_build, "build_native", lambda: None)
        return log, lib, nowait
    return install


def test_both_libraries(stand_in):
    log, lib, nowait = stand_in("nothing")
    assert akvq_build.build() == str(lib)
    assert lib.read_text() == nowait.read_text() == "new\n"
    compiled = [line for line in log.read_text().splitlines() if " -c " in line]
    assert sum("AKVQ_ONCE_POLLS=0" in line for line in compiled) == 1 and len(compiled) == len(akvq_build.SOURCES) + 1
    links = [line for line in log.read_text().splitlines() if "-shared" in line]
    assert [("akvq_select_nowait.o" in line, "akvq_select.o" in line) for line in links] == [(False, True), (True, False)]


@pytest.mark.parametrize("fail", ["akvq_select_nowait.o", "akvq_decode.o"])
def test_a_failure_is_told_and_leaves_no_old_library(stand_in, fail):
    log, lib, nowait = stand_in("-c*" + fail)
    with pytest.raises(RuntimeError, match="what went wrong"):
        akvq_build.build()
    assert not os.path.exists(lib) and not os.path.exists(nowait)
