"""The binding's stream query after a fork, on the host: once a call has found the raw queries of the
current stream, a forked child still goes through torch's own query first, which refuses a GPU that
the parent has used.  Stand-ins play the GPU, so none is needed."""
import os

import pytest

torch = pytest.importorskip("torch")
ntt = pytest.importorskip("paper_2012_01968_amd")


def test_forked_child_asks_torch_first(monkeypatch):
    class FakeStream:
        cuda_stream = 7

    monkeypatch.setattr(torch.cuda, "current_stream", lambda: FakeStream())
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 7, raising=False)
    monkeypatch.setattr(ntt, "_current_stream", ntt._first_current_stream)
    assert ntt._stream(None) == 7 and ntt._stream(None) == 7      # the second through the raw queries

    def refuse():
        raise RuntimeError("the parent has used the GPU")

    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    assert ntt._stream(None) == 7                                 # the parent keeps its queries
    pid = os.fork()
    if pid == 0:
        try:
            ntt._stream(None)
            os._exit(1)                                           # a child that takes the parent's stream
        except RuntimeError:
            os._exit(0)
        except BaseException:
            os._exit(2)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
