"""A build leaves nothing but the library in the source tree, also when it is
interrupted: the compiler writes an object through a temporary beside it, which
stays behind when the compiler is killed."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _csrc():
    return sorted(os.listdir(os.path.join(ROOT, "paper_2511_02700_amd", "csrc")))


def test_no_compiler_output_is_tracked():
    try:
        r = subprocess.run(["git", "ls-files"], cwd=ROOT, capture_output=True, text=True, timeout=60)
    except OSError:
        pytest.skip("git not installed")
    if r.returncode != 0:
        pytest.skip("not a git checkout")
    assert [f for f in r.stdout.split("\n") if f.endswith((".o", ".so", ".tmp"))] == []


@pytest.mark.parametrize("interrupted", [False, True])
def test_build_leaves_the_sources_alone(monkeypatch, tmp_path, interrupted):
    from paper_2511_02700_amd import build as b
    lib = tmp_path / "lib.so"
    monkeypatch.setattr(b, "LIB", str(lib))

    def compiler(cmd, check):
        out = cmd[cmd.index("-o") + 1]
        with open(out + ".tmp-of-the-compiler", "w"):
            pass
        if interrupted and "-c" in cmd:
            raise subprocess.CalledProcessError(-9, cmd)
        os.rename(out + ".tmp-of-the-compiler", out)

    monkeypatch.setattr(b.subprocess, "run", compiler)
    before = _csrc()
    try:
        if interrupted:
            with pytest.raises(subprocess.CalledProcessError):
                b.build()
            assert not lib.exists()
        else:
            assert b.build() == str(lib) and lib.exists()
        assert _csrc() == before
    finally:
        for f in set(_csrc()) - set(before):
            os.remove(os.path.join(ROOT, "paper_2511_02700_amd", "csrc", f))
