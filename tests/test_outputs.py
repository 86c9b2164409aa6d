"""The output tensors that the binding makes in one step are what torch.empty gives."""
import pytest
import torch

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
