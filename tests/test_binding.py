"""The product calls through the C extension: the arguments, defaults, results and errors of the ctypes functions."""
import inspect

import pytest

import paper_2003_06324_amd as g
from paper_2003_06324_amd import gemm


def _general(name):
    """The ctypes function behind an entry point: any keyword argument goes there."""
    return lambda *a, **k: getattr(g, name)(*a, **dict({"stream": None}, **k))


@pytest.mark.parametrize("name", gemm.PRODUCTS)
def test_plain_and_general_calls_agree(name):
    fn, general = getattr(g, name), _general(name)
    g.load_library()
    assert fn is getattr(gemm, name)
    assert [p for p in inspect.signature(fn).parameters] == ["M", "N", "K", "A", "layoutA", "lda", "B", "layoutB", "ldb", "C", "layoutC",
                                                             "ldc", "stream", "check"]
    empty = (0, 5, 7, None, 0, 0, 16, 1, 0, None, 0, 0)
    assert fn(*empty) == general(*empty) == 0 and fn(*empty, 0, True) == 0
    assert g.last_config().endswith(" empty")
    bad = (4, 4, 4, 16, 7, 0, 16, 0, 0, 16, 0, 0)          # no such layout
    for call in (fn, general):
        with pytest.raises(g.GemmError) as e:
            call(*bad)
        assert e.value.status == -1
    assert fn(*bad, None, False) == general(*bad, check=False) == fn(*bad, stream=None, check=0) == -1
    null = (4, 4, 4, 0, 0, 0, 16, 0, 0, 16, 0, 0)          # a null operand
    assert fn(*null, 0, False) == -1
    for args in (bad[:11], (4.0,) + bad[1:], bad[:3] + ("x",) + bad[4:], bad[:3] + (1.5,) + bad[4:], bad[:4] + ("row",) + bad[5:]):
        errors = []
        for call in (fn, general):
            with pytest.raises(Exception) as e:
                call(*args)
            errors.append(e.type)
        assert errors[0] is errors[1], (args, errors)
    with pytest.raises(TypeError):
        fn(*bad, None, True, 1)


def test_an_object_with_a_data_pointer_and_its_errors():
    class Owner:
        def __init__(self, p):
            self.p = p

        def data_ptr(self):
            if self.p is None:
                raise KeyError("gone")
            return self.p

    ok = (0, 0, 0, Owner(16), 0, 0, Owner(0), 0, 0, Owner(16), 0, 0)
    assert g.gemm_f32(*ok) == 0
    with pytest.raises(KeyError):
        g.gemm_f32(0, 0, 0, Owner(None), 0, 0, None, 0, 0, None, 0, 0)


def test_whole_numbers_beyond_the_c_types_go_the_general_way():
    big = (2 ** 63, 1, 1, 16, 0, 0, 16, 0, 0, 16, 0, 0)
    assert g.gemm_f32(*big, None, False) == _general("gemm_f32")(*big, check=False)
    assert g.gemm_f32(True, 0, True, 16, False, 0, 16, 0, 0, 16, 0, 0) == 0


@pytest.mark.parametrize("compiler", ["false", "/no/such/compiler"])
def test_the_library_is_built_without_a_compiler_for_the_extension(monkeypatch, tmp_path, compiler):
    from paper_2003_06324_amd import build
    built = []
    monkeypatch.setenv("CXX", compiler)
    monkeypatch.setattr(build, "OBJDIR", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "ext.so"))
    monkeypatch.setattr(build, "_compile", lambda src, force: built.append(src) or src)
    monkeypatch.setattr(build, "HIPCC", "true")
    monkeypatch.setattr(build.os, "replace", lambda a, b: open(b, "w").close())
    with pytest.warns(UserWarning, match="extension was not built"):
        assert build.build() == str(tmp_path / "lib.so")
    assert built == build.sources()
