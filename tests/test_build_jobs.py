"""CPU: the build's compile jobs run side by side; no two of them write into one folder (kept temporaries are named after the source, which the
jobs of the index widths share)."""
from pathlib import Path

from paper_2506_12038_amd import build


def test_every_job_has_a_folder_of_its_own(monkeypatch, tmp_path):
    commands = []
    monkeypatch.setattr(build, "BUILD", tmp_path / "objects")
    monkeypatch.setattr(build, "LIB", tmp_path / "liblcd.so")
    monkeypatch.setattr(build.os, "replace", lambda a, b: None)
    monkeypatch.setattr(build.subprocess, "check_call", lambda cmd, **kw: commands.append((cmd, kw.get("cwd"))))
    build.build_library(keep_asm=True)
    jobs = [(Path(cmd[cmd.index("-o") + 1]).parent, Path(cwd)) for cmd, cwd in commands if "-c" in cmd]
    assert len(jobs) == len(build.SOURCES) + 2 * len(build.EACH_WIDTH)
    assert len({folder for folder, _ in jobs}) == len(jobs)
    assert all(folder == cwd and folder.is_dir() for folder, cwd in jobs)
    linked = [Path(a) for cmd, _ in commands if "-shared" in cmd for a in cmd if a.endswith(".o")]
    assert sorted(o.parent for o in linked) == sorted(folder for folder, _ in jobs)
