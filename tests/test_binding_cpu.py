"""What fa2_fwd refuses before any launch, and what it does without its native call, without a GPU: stand-ins for device tensors, which have no memory."""
import pytest
import torch

import paper_2312_11918_amd as fa2
from paper_2312_11918_amd import binding


class StandIn:
    def __init__(self, shape, dtype, device):
        self.shape, self.dtype, self.device = torch.Size(shape), dtype, torch.device(device)

    is_cuda = property(lambda self: self.device.type == "cuda")

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True


@pytest.fixture
def launches(monkeypatch):
    seen = []
    monkeypatch.setattr(binding, "_launch", lambda *args: seen.append(args) or fa2.FA2_OK)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    return seen


def _call(q="cuda:0", k="cuda:0", v="cuda:0", out="cuda:0", lse="cuda:0"):
    half = [StandIn((1, 128, 2, 64), torch.float16, x) for x in (q, k, v, out)]
    return fa2.fa2_fwd(*half[:3], 0.125, out=half[3], lse=StandIn((1, 2, 128), torch.float32, lse))


def test_tensors_of_one_device_are_launched(launches):
    _call()
    assert len(launches) == 1


@pytest.mark.parametrize("which", ["k", "v", "out", "lse"])
@pytest.mark.parametrize("device", ["cpu", "cuda:1"])
def test_a_tensor_elsewhere_is_refused_before_a_launch(launches, which, device):
    with pytest.raises(ValueError):
        _call(**{which: device})
    assert not launches


def _no_file(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_TORCH_PATH", str(tmp_path / "_fa2_torch.so"))


def _not_a_library(monkeypatch, tmp_path):
    (tmp_path / "_fa2_torch.so").write_bytes(b"text")
    _no_file(monkeypatch, tmp_path)


def _other_torch(monkeypatch, tmp_path):
    monkeypatch.setattr(torch, "__version__", "1.0.0")


@pytest.mark.parametrize("lacking", [_no_file, _not_a_library, _other_torch])
def test_calls_without_the_native_call_go_the_python_path(launches, monkeypatch, tmp_path, lacking):
    monkeypatch.setattr(binding, "_forward", None)
    lacking(monkeypatch, tmp_path)
    with pytest.warns(RuntimeWarning, match="_fa2_torch.so"):
        _call()
    _call()   # (says so once)
    assert len(launches) == 2


def test_the_native_call_loads(monkeypatch):
    monkeypatch.setattr(binding, "_forward", None)
    assert binding._load_forward() is not binding._leave_to_python
