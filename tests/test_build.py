"""The build script itself: what it says when a source does not compile."""
import pytest

from paper_2312_17482_amd import build


@pytest.mark.parametrize("which", ["marshal", "kernels"])
def test_a_source_that_does_not_compile_is_named(tmp_path, monkeypatch, which):
    csrc = tmp_path / "csrc"
    csrc.mkdir()
    (csrc / "marshal.cpp").write_text("int whole;" if which == "kernels" else "no source")
    (csrc / "k.hip").write_text("no source" if which == "kernels" else "int whole;")
    monkeypatch.setattr(build, "CSRC", str(csrc))
    monkeypatch.setattr(build, "LIBDIR", str(tmp_path / "lib"))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "lib" / "_mosaic_marshal.so"))
    name = str(csrc / ("marshal.cpp" if which == "marshal" else "k.hip"))
    with pytest.raises(RuntimeError) as e:
        build.build(verbose=False)
    assert str(e.value).startswith("compiling %s failed" % name)
