"""What the build does where one of its two compilers fails, with stand-ins for the compilers (nothing is compiled)."""
import importlib.util
import os
import stat
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def build(tmp_path, monkeypatch):
    """build(library compiler's exit status, module compiler's): the build script on outputs of its own, an old module among them."""
    def compiler(name, status):
        path = tmp_path / name
        path.write_text(f'#!{sys.executable}\nimport sys\nprint("{name} was here")\nif {status} == 0:\n'
                        f'    open(sys.argv[sys.argv.index("-o") + 1], "w").write("{name}")\nsys.exit({status})\n')
        path.chmod(path.stat().st_mode | stat.S_IXUSR)
        return str(path)

    def run(library, module):
        spec = importlib.util.spec_from_file_location("build_under_test", os.path.join(ROOT, "paper_1802_06905_amd", "build.py"))
        script = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(script)
        script.HIPCC, script.LIB, script.TORCH_LIB = compiler("hipcc", library), str(tmp_path / "lib.so"), str(tmp_path / "module.so")
        monkeypatch.setenv("CXX", compiler("g++", module))
        (tmp_path / "module.so").write_text("old")
        return script.build(), tmp_path
    return run


def test_both_compile(build):
    lib, where = build(0, 0)
    assert lib == str(where / "lib.so") and (where / "lib.so").read_text() == "hipcc" and (where / "module.so").read_text() == "g++"


def test_the_library_is_built_without_its_module(build):
    """The binding works without the module; an old one, made for another library, must not stay beside the new one."""
    with pytest.warns(RuntimeWarning, match="g\\+\\+ was here"):
        lib, where = build(0, 1)
    assert (where / "lib.so").read_text() == "hipcc" and not (where / "module.so").exists()


@pytest.mark.parametrize("module", [0, 1])
def test_a_failure_of_hipcc_is_what_is_reported(build, module):
    with pytest.raises(RuntimeError, match="hipcc was here"):
        build(1, module)


def test_the_compiler_may_be_named_without_its_folder(build, tmp_path, monkeypatch):
    """HIPCC=hipcc: the runtime's headers lie beside the compiler that PATH finds."""
    build(0, 0)
    import paper_1802_06905_amd.build as script
    (tmp_path / "bin").mkdir()
    (tmp_path / "hipcc").rename(tmp_path / "bin" / "hipcc")
    monkeypatch.setenv("PATH", str(tmp_path / "bin"), prepend=os.pathsep)
    monkeypatch.setattr(script, "HIPCC", "hipcc")
    assert str(tmp_path / "include") in script.torch_command()


def test_the_module_refuses_another_library_interface():
    from paper_1802_06905_amd import binding
    good = binding._native_interface()
    binding._native.setup(*good)
    for version, size in ((good[0] + 1, good[1]), (good[0], good[1] + 8)):
        with pytest.raises(ImportError):
            binding._native.setup(version, size, *good[2:])
    assert binding._native.conv() == -1
