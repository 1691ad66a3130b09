"""The current stream's handle without torch's private names: the binding falls
back to the public way, and either gives the same handle."""
import pytest

torch = pytest.importorskip("torch")
drt = pytest.importorskip("paper_2109_08219_amd")


class Cuda:
    def __init__(self):
        self.inits = 0

    def is_initialized(self):
        return self.inits > 0

    def init(self):
        self.inits += 1

    def current_stream(self):
        return type("S", (), {"cuda_stream": 77})()


def test_falls_back_to_the_public_name(monkeypatch):
    fake = type("T", (), {"cuda": Cuda(), "_C": object()})()
    monkeypatch.setattr(drt, "_torch", lambda: fake)
    assert drt._stream(None) == 77 and fake.cuda.inits == 1
    assert drt._stream(type("S", (), {"cuda_stream": 5})()) == 5


@pytest.mark.gpu
def test_both_ways_agree():
    s = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), s):
        with torch.cuda.stream(stream):
            assert drt._stream(None) == torch.cuda.current_stream().cuda_stream == stream.cuda_stream
