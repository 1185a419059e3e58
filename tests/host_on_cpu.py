"""csrc/host.cpp built for tensors in ordinary memory, and a stand-in for the library, so that the native marshalling of the
binding's calls can be looked at without a GPU."""
import ctypes
import importlib.machinery
import importlib.util
import os
import shutil

import pytest
import torch

from paper_2503_03588_amd import binding as pa
from paper_2503_03588_amd import build as b

STREAM = 0x5150

# Beside the module: how many allocations were made with the GIL held, and without, since the last look.
WATCH = """
namespace {
struct watching : c10::Allocator {
  c10::Allocator* real;
  int held = 0, released = 0;
  c10::DataPtr allocate(size_t n) override { ++(PyGILState_Check() ? held : released); return real->allocate(n); }
  c10::DeleterFnPtr raw_deleter() const override { return real->raw_deleter(); }
  void copy_data(void* to, const void* from, size_t n) const override { real->copy_data(to, from, n); }
} watch;
}
extern "C" void watch_allocations(int on) {
  if (on) { watch.real = c10::GetAllocator(c10::kCPU); watch.held = watch.released = 0; c10::SetAllocator(c10::kCPU, &watch, 200); }
  else c10::SetAllocator(c10::kCPU, watch.real, 200);
}
extern "C" int allocations_with_gil() { return watch.held; }
extern "C" int allocations_without_gil() { return watch.released; }
"""


@pytest.fixture(scope="session")
def host_cpu(tmp_path_factory):
    if not shutil.which(os.environ.get("CXX") or "g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("host")
    src = d / "host_cpu.cpp"
    src.write_text(f'#define POWATTN_HOST_DEVICE at::kCPU\n#include "{os.path.join(b.CSRC, "host.cpp")}"\n' + WATCH)
    out = b.build_host(verbose=False, src=str(src), out=str(d / "_host.so"))
    loader = importlib.machinery.ExtensionFileLoader("host_cpu._host", out)
    module = importlib.util.module_from_spec(importlib.util.spec_from_loader("host_cpu._host", loader))
    loader.exec_module(module)
    return module


class StandIn:
    """What the binding sees as the library: the sizes come from the real one, every call is written down and answered with
    the status at the head of `answers` (0 when there is none)."""

    def __init__(self):
        self.seen, self.answers = [], []
        real = pa.lib()
        for name in pa.EXPORTS:
            f = getattr(real, name)
            if name[len("powattn_"):] not in pa._NATIVE_ENTRY_POINTS or f.restype is not ctypes.c_int or "bytes" in name:
                setattr(self, name, f)
                continue
            setattr(self, name, ctypes.CFUNCTYPE(ctypes.c_int, *f.argtypes)(self._called(name)))
        self.powattn_num_blocks, self.powattn_max_k = real.powattn_num_blocks, real.powattn_max_k

    def _called(self, name):
        def f(pattern, *args):
            c = pattern.contents
            self.seen.append((name, (c.block, c.window, c.sink, c.flags), args))
            return self.answers.pop(0) if self.answers else pa.OK
        return f

    def bind(self, host):
        host.bind(*(ctypes.cast(getattr(self, "powattn_" + n), ctypes.c_void_p).value for n in pa._NATIVE_ENTRY_POINTS),
                  torch.Tensor, lambda: 0, lambda device: STREAM, pa._check)


@pytest.fixture
def stand_in(host_cpu, monkeypatch):
    """The binding with the stand-in below it and the CPU build of the native marshalling in use."""
    fake = StandIn()
    fake.bind(host_cpu)
    monkeypatch.setattr(pa, "lib", lambda: fake)
    monkeypatch.setattr(pa, "_stream", lambda stream=None: STREAM)
    monkeypatch.setattr(pa, "_native", host_cpu)
    return fake
