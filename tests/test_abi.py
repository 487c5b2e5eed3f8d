"""The C-ABI library loads and exports every function include/oxy.h declares.  No GPU,
no compute calls."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2603_14371_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "oxy.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(oxy_[a-z_]+)\s*\(", text)))


def test_every_declared_function_is_exported_and_bound():
    names = _declared()
    assert "oxy_pool_create" in names and "oxy_prefix_append" in names
    assert "oxy_stream_append" in names and "oxy_mixed_attention" in names
    lib = ctypes.CDLL(binding.LIB_PATH)
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(binding.EXPORTS) == names
    for name in names:
        assert callable(getattr(binding, name)), name
    assert binding.oxy_version() == 1


def test_signatures_carry_no_framework_types():
    text = open(os.path.join(ROOT, "include", "oxy.h")).read()
    assert "torch" not in text and "at::" not in text and "#include <hip" not in text


def test_invalid_configs_are_rejected_without_a_device():
    cfg = binding.make_config(2, 8, flags=binding.POOL_HOST_ONLY, head_dim=128)
    assert binding.oxy_kv_bytes(cfg) == 0
    try:
        binding.oxy_pool_create(cfg)
        assert False
    except binding.OxyError as e:
        assert e.code == binding.ERR_INVALID_ARG
    cfg = binding.make_config(2, 8)                # not host-only but no device buffers
    try:
        binding.oxy_pool_create(cfg)
        assert False
    except binding.OxyError as e:
        assert e.code == binding.ERR_INVALID_ARG
    cfg = binding.make_config(18, 8192)
    assert binding.oxy_kv_bytes(cfg) == 18 * 8192 * 16384


@pytest.mark.parametrize("values", [
    [], [0], [5, -1, 2**63 - 1, -2**63], (7, 8), [True, 2], [np.int64(4), 5], [1.0, 2], np.arange(3),
    np.arange(8, dtype=np.int32)[::3], [2**63], [1, None], ["1"],
], ids=str)
@pytest.mark.parametrize("times", [1, 20, 48])
@pytest.mark.parametrize("native", [True, False], ids=["libmarshal", "liboxy_alone"])
def test_integer_sequences_reach_the_library_as_numpy_converts_them(values, native, times, monkeypatch):
    """oxy_gather_kv takes any sequence of integers; a long list of plain ints is converted natively
    where libmarshal.so is there."""
    values = np.tile(values, times) if isinstance(values, np.ndarray) else values * times
    monkeypatch.setattr(binding, "_marshal_lib", None)
    if native and not os.path.exists(binding.MARSHAL_PATH):
        pytest.skip("libmarshal.so is not built here")
    if not native:
        monkeypatch.setattr(binding, "MARSHAL_PATH", "/nowhere/libmarshal.so")
    assert bool(binding._marshal()) == native
    calls = []
    if native:
        class Counting:
            def oxy_ints_of_list(self, *args):
                calls.append(args)
                return lib.oxy_ints_of_list(*args)
        lib = binding._marshal()
        monkeypatch.setattr(binding, "_marshal_lib", Counting())
    try:
        want = np.ascontiguousarray(values, dtype=np.int64)
    except (TypeError, ValueError, OverflowError) as e:
        with pytest.raises(type(e)):
            binding._i64(values)
        return
    arr, ptr, n = binding._i64(values)
    assert len(calls) == (native and type(values) is list and n >= 48)
    assert n == len(want) and [int(x) for x in arr] == want.tolist()
    assert [ctypes.c_int64.from_address(ptr + 8 * i).value for i in range(n)] == want.tolist()


@pytest.mark.parametrize("missing", ["compiler", "headers"])
def test_the_library_builds_without_python_headers_or_a_host_compiler(missing, monkeypatch, tmp_path):
    from paper_2603_14371_amd import build
    built = []
    monkeypatch.setattr(build, "_compile", lambda compiler, flags, sources, target, verbose: built.append(target))
    monkeypatch.setattr(build, "MARSHAL_LIB", str(tmp_path / "libmarshal.so"))
    (tmp_path / "libmarshal.so").write_text("of an earlier build")
    if missing == "compiler":
        monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    else:
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_library() == build.LIB
    assert built == [build.LIB, build.PROBE_LIB] and not os.path.exists(build.MARSHAL_LIB)


LIST = "const int32_t part_off, const float scale, const LateArgs)"


@pytest.mark.parametrize("params,builds", [
    (LIST, True),
    (LIST.replace("int32_t", "int64_t"), False),                       # the last argument lies 8 bytes further on
    (LIST.replace("const float scale, const LateArgs", "const LateArgs, const float scale"), False),
], ids=["as_it_is", "wider", "reordered"])
def test_last_argument_of_the_work_items_is_where_it_is_read(tmp_path, params, builds):
    """Work items read their last argument at an offset of their own: another parameter list does not build."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    csrc = os.path.join(ROOT, "paper_2603_14371_amd", "csrc")
    text = open(os.path.join(csrc, "oxy_kernels.hip")).read()
    assert text.count(LIST) == 1
    src = tmp_path / "kernels.hip"
    src.write_text(text.replace(LIST, params))
    res = subprocess.run([hipcc, "-fsyntax-only", "--cuda-device-only", "-std=c++17", "--offload-arch=gfx950",
                          "-I" + csrc, str(src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert (res.returncode == 0) == builds, res.stdout[-2000:]
    assert ("take_late reads" in res.stdout) == (not builds), res.stdout[-2000:]
