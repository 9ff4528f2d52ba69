"""What the compiler makes of the device code, without a GPU: no warnings (and a build shows those there are), and the
requests into LDS that are written out in assembly keep the distances that the hardware asks for (the compiler does
not look inside)."""
import os
import re
import subprocess

import pytest

from paper_2411_15785_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")


@pytest.fixture(scope="module")
def prefill_isa(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "prefill.s")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--offload-device-only", os.path.join(build.CSRC, "bct_prefill.hip"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stderr, open(out).read()


def test_device_compile_has_no_warnings(prefill_isa):
    warnings = [l for l in prefill_isa[0].splitlines() if "warning:" in l]
    assert not warnings, f"{len(warnings)} warnings, the first: {warnings[0]}"


def test_build_shows_the_compilers_warnings(tmp_path, monkeypatch, capsys):
    cc = tmp_path / "cc"
    cc.write_text("#!/bin/sh\n"
                  "echo \"'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)\" >&2\n"
                  "echo 'x.hip:3:5: warning: unused variable' >&2\n")
    cc.chmod(0o755)
    monkeypatch.setattr(build, "HIPCC", str(cc))
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    build._compile("x.hip", verbose=False)
    assert capsys.readouterr().out == "x.hip:3:5: warning: unused variable\n"


# A load must not come within 5 wait states of a vector instruction's write of its scalar base, nor within 1 of a write
# of m0.  What stands before an assembly block is the compiler's choice, so the block itself writes the base, by a
# scalar instruction (none needed from there on), and has an instruction between its start and the load.
def test_lds_requests_keep_their_wait_states(prefill_isa):
    blocks = [[l.strip() for l in b.splitlines() if l.strip()]
              for b in re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", prefill_isa[1], flags=re.S)]
    requests = [b for b in blocks if any(l.startswith("global_load_lds") for l in b)]
    assert len(requests) > 100
    for b in requests:
        assert [l.startswith("global_load_lds") for l in b] == [False] * (len(b) - 1) + [True], b
        assert len(b) >= 2 and not any(re.search(r"\bm0\b", l) for l in b), f"m0 is an operand of the block: {b}"
        base = re.search(r"s\[\d+:\d+\]", b[-1])
        if base:
            copy = re.fullmatch(r"s_mov_b64 (s\[\d+:\d+\]), s\[\d+:\d+\]", b[-2])
            assert copy and copy[1] == base[0], b
