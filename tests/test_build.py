"""What the build needs: hipcc for the library, headers beyond that only for the Python extension (nothing is compiled here)."""
import pytest

from paper_2403_12422_amd import binding, build


@pytest.fixture
def commands(monkeypatch, tmp_path):
    """Commands that build() would run; those of the extension fail as they do without its headers."""
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        if any("jf_python" in a for a in cmd):
            raise RuntimeError("Python.h: no such file")

    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path))
    monkeypatch.setattr(build, "EXT", str(tmp_path / "_native.so"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libjetfire.so"))
    return ran


def test_library_is_linked_where_the_extension_cannot_be_built(commands):
    with pytest.raises(RuntimeError, match="libjetfire.so is built"):
        build.build()
    assert commands[-1][-1] == build.LIB and "-shared" in commands[-1]


def test_library_alone(commands):
    assert build.build(extension=False) == build.LIB
    assert not any("jf_python" in a or "torch" in a for cmd in commands for a in cmd)


def test_hipcc_is_the_only_compiler(commands, monkeypatch):
    monkeypatch.setenv("HIPCC", "/somewhere/hipcc")
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: commands.append(cmd))
    build.build()
    assert {cmd[0] for cmd in commands} == {"/somewhere/hipcc"}


def test_missing_extension_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_ext", None)
    monkeypatch.setattr(binding, "_EXT_PATH", str(tmp_path / "_native.so"))
    with pytest.raises(binding.JetfireError, match="load_library"):
        binding.jf_gelu_q(None, None)


def test_digest_is_of_the_flags_too(monkeypatch):
    """A recorded profile counts as one of the present kernels by this digest, and the flags make other kernels of the same sources."""
    before = build.source_digest()
    assert build.source_digest() == before
    assert any("preload-count" in flag for flag in build.HIPCC_FLAGS)
    monkeypatch.setattr(build, "HIPCC_FLAGS", [flag.replace("preload-count=14", "preload-count=13") for flag in build.HIPCC_FLAGS])
    assert build.source_digest() != before
