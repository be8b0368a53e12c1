"""CPU-only checks of the binding itself."""
import importlib.util
import os
import struct

import pytest
import torch

from paper_2406_09904_amd import binding


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_handle_without_torchs_private_names(monkeypatch, missing):
    """A torch without one of them: the handle comes from torch.cuda.current_stream()."""
    class Stream:
        cuda_stream = 0x1234

    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream if device == 3 else None)
    spec = importlib.util.spec_from_file_location("binding_without_" + missing, binding.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module._stream() == 0x1234
    assert module._raw_stream(module._device()) == 0x1234


@pytest.mark.parametrize("kind", ["missing", "damaged", "another module's"])
def test_library_without_a_fitting_extension(monkeypatch, tmp_path, kind):
    """Only the linear calls' marshalling is in the extension: without one that can be loaded the library is still whole, beside a GPU too."""
    path = tmp_path / "_qqq_call.so"
    if kind == "damaged":
        path.write_bytes(b"\x7fELF nothing")
    elif kind == "another module's":
        import _struct
        path.write_bytes(open(_struct.__file__, "rb").read() if getattr(_struct, "__file__", None) else open(binding.LIB_PATH, "rb").read())
    spec = importlib.util.spec_from_file_location("paper_2406_09904_amd.binding_alone", binding.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(module, "_call_path", lambda: str(path))
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        module.lib()
    assert module._native_linear is module._no_native
    assert module.qqq_packed_w4_bytes(4096, 4096) == 4096 * 4096 // 2


def test_extension_is_the_present_torchs():
    """The file's name carries the torch and the interpreter that it was built against."""
    from paper_2406_09904_amd import build
    import sysconfig
    name = os.path.basename(build.call_path())
    assert torch.__version__ in name and sysconfig.get_config_var("SOABI") in name
    binding.lib()
    assert binding._native_linear is not binding._no_native


def test_extension_has_no_thread_local_variables():
    """One that nothing reads would slow down every access to torch's and HIP's (glibc 2.35: the thread's table of modules counts as out of date until
    the newest module's entry is asked for), a microsecond for each of the library's calls."""
    from paper_2406_09904_amd import build
    image = open(build.call_path(), "rb").read()
    at, size, count = struct.unpack_from("<Q", image, 32)[0], *struct.unpack_from("<HH", image, 54)
    kinds = [struct.unpack_from("<I", image, at + size * i)[0] for i in range(count)]
    assert image[:5] == b"\x7fELF\x02" and 1 in kinds           # PT_LOAD
    assert 7 not in kinds                                         # PT_TLS
