"""What the build compiles again.  No GPU needed."""
import os


def test_a_changed_header_rebuilds_the_binding(monkeypatch, tmp_path):
    from paper_2601_16991_amd import build
    header = tmp_path / "changed.hpp"
    header.write_text("")
    os.utime(header, (1 << 40, 1 << 40))   # newer than every object
    monkeypatch.setattr(build, "_headers", lambda: [str(header)])
    todo, objects = build._compile_commands(only_changed=True)
    assert build.BINDING_SRC in [cmd[-1] for cmd in todo]
    assert [cmd[-1] for cmd in todo if cmd[-1] != build.BINDING_SRC] == build.sources() and len(objects) == len(build.sources())
