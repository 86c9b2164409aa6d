"""The output tensors that the binding makes in one step are what torch.empty gives."""
import os
import sys
import sysconfig
import threading
import time

import pytest
import torch
from torch.overrides import TorchFunctionMode

from paper_2506_05632_amd import binding


def test_what_is_not_a_list_of_tensors_is_refused():
    binding.load()
    for args in ((), (-1, (torch.int32, 3)), (0, [torch.int32, 3]), (0, ("int32", 3)), (0, ()), (0, (torch.int32, 3.5)),
                 (0, (torch.int32, 1, 1, 1, 1, 1)), ("cuda:0", (torch.int32, 3))):
        with pytest.raises((TypeError, ValueError)):
            binding._empties(*args)


@pytest.mark.gpu
def test_tensors_of_their_own():
    binding.load()
    dev = torch.device("cuda:0")
    specs = {"a": (torch.int32, 5, 3), "b": (torch.uint8, 7), "c": (torch.float64, 0, 4), "d": (torch.float32,)}
    made = binding._new(dev, specs)
    for name, (dtype, *size) in specs.items():
        t = made[name]
        assert t.dtype == dtype and tuple(t.shape) == tuple(size) and t.device == dev
        assert t.is_contiguous() and t.storage_offset() == 0 and t.untyped_storage().nbytes() >= t.nbytes
        assert not t.requires_grad
    assert len({t.untyped_storage().data_ptr() for t in made.values() if t.numel()}) == 3
    with pytest.raises(RuntimeError):
        binding._empties(0, (torch.int32, -3))


class _OnTheHost(TorchFunctionMode):
    def __init__(self):
        super().__init__()
        self.seen = []

    def __torch_function__(self, func, types, args=(), kwargs=None):
        kwargs = dict(kwargs or {})
        if func is torch.empty:
            self.seen.append((tuple(args[0]), kwargs.get("dtype"), kwargs.pop("device")))
        return func(*args, **kwargs)


def test_a_mode_that_overrides_functions_sees_the_outputs():
    binding.load()
    dev = torch.device("cuda:0")
    with _OnTheHost() as mode:
        made = binding._new(dev, {"a": (torch.int32, 5, 3), "b": (torch.float64,)})
    assert mode.seen == [((5, 3), torch.int32, dev), ((), torch.float64, dev)]
    assert made["a"].shape == (5, 3) and made["a"].dtype == torch.int32 and made["b"].shape == ()


def test_the_module_belongs_to_this_torch_and_this_python(monkeypatch):
    name = os.path.basename(binding.OUTPUTS_PATH)
    assert torch.__version__ in name and name.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert os.path.exists(binding.OUTPUTS_PATH)
    # one of another torch is not there under this name: the library loads, and torch.empty makes the tensors
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_empties", None)
    monkeypatch.setattr(binding, "OUTPUTS_PATH", binding.OUTPUTS_PATH + ".other")
    assert binding.load() is not None and binding._empties is None
    made = binding._new(torch.device("cpu"), {"a": (torch.uint8, 4), "b": (torch.float32, 2, 0, 3)})
    assert made["a"].shape == (4,) and made["b"].shape == (2, 0, 3) and made["a"].dtype == torch.uint8


@pytest.mark.gpu
def test_other_threads_run_while_the_tensors_are_allocated():
    binding.load()
    torch.cuda.empty_cache()
    interval = sys.getswitchinterval()
    ran, ready = [], threading.Event()

    def other():
        ready.set()
        time.sleep(0.05)
        ran.append(True)

    try:
        sys.setswitchinterval(1000.0)  # (nobody is made to give Python's lock up)
        thread = threading.Thread(target=other)
        thread.start()
        ready.wait()
        until = time.perf_counter() + 0.2
        while time.perf_counter() < until:
            pass
        before = list(ran)  # (the other thread has waited for the lock for 0.15 s)
        made = binding._empties(0, *[(torch.uint8, (1 << 30) + n) for n in range(7)])  # 0.4 ms each from the device
        after = list(ran)
    finally:
        sys.setswitchinterval(interval)
    thread.join()
    assert before == [] and after == [True]
    del made
    torch.cuda.empty_cache()
