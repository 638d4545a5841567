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


def test_kernels_on_2of4_weights_have_no_scratch(tmp_path):
    """The small-batch kernel there is bounded to 128 registers, so that two of its workgroups fit a CU: a value too many that is kept through
    its stream goes to memory and back, 5 to 20 % of a call."""
    import re
    import subprocess
    from paper_2601_16991_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    text = subprocess.run([hipcc, *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-c",
                           "-Rpass-analysis=kernel-resource-usage", "-o", str(tmp_path / "kernels.o"), os.path.join(build.CSRC, "salr_linear_2of4.hip")],
                          capture_output=True, text=True, check=True, timeout=300).stderr
    scratch = dict(zip(re.findall(r"Function Name: (\S+)", text), map(int, re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", text))))
    assert sum("linear_2of4_stream_kernel" in name for name in scratch) == 2
    assert not {name: n for name, n in scratch.items() if n}
