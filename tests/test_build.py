"""An incremental build compiles what its objects are no longer the result of (the compiler is replaced by one that notes its
command and writes an empty object)."""
import os
import time

from paper_2506_03887_amd import build as B


def test_incremental_builds(tmp_path, monkeypatch):
    src, obj = tmp_path / "csrc", tmp_path / "obj"
    src.mkdir()
    for name in (*B.SOURCES, "one.hpp"):
        (src / name).write_text("")
    old = time.time() - 100
    for f in src.iterdir():
        os.utime(f, (old, old))
    header = tmp_path / "include"
    header.mkdir()
    (header / "pre3.h").write_text("")
    os.utime(header / "pre3.h", (old, old))
    (tmp_path / "pkg").mkdir()
    for name, value in (("CSRC", src), ("OBJ", obj), ("LIB", tmp_path / "lib.so"), ("HERE", tmp_path / "pkg")):
        monkeypatch.setattr(B, name, str(value))
    ran, fails = [], []

    def run(cmd):
        if any(f in cmd[-1] for f in fails):
            raise RuntimeError("refused")
        open(cmd[cmd.index("-o") + 1], "w").close()
        if "-c" in cmd:
            ran.append(os.path.basename(cmd[-1]))
        return ""

    def compiled(**kw):
        ran.clear()
        B.build(**kw)
        return sorted(ran)

    monkeypatch.setattr(B, "_run", run)
    everything = sorted(B.SOURCES)
    assert compiled(incremental=True) == everything                          # nothing there yet
    assert compiled(incremental=True) == [] and compiled() == everything and compiled(incremental=True) == []
    os.utime(src / "api.cpp", (time.time() + 5,) * 2)
    assert compiled(incremental=True) == ["api.cpp"]
    os.utime(src / "api.cpp", (old, old))
    monkeypatch.setattr(B, "FLAGS", B.FLAGS + ["-DOTHER"])
    assert compiled(incremental=True) == everything                          # other flags: no old object is kept
    assert compiled(incremental=True) == []
    monkeypatch.setattr(B, "FLAGS", B.FLAGS + ["-DMORE"])
    fails.append("api.cpp")
    try:
        compiled(incremental=True)
    except RuntimeError:
        fails.clear()
    assert compiled(incremental=True) == everything                          # a build that failed left objects of both kinds
