"""Plan.execute without a stream argument runs on torch's current stream: the
default one, a side stream, one made current inside another, and each thread's
own."""
import threading

import pytest

from paper_2604_00567_amd import binding

pytestmark = pytest.mark.gpu


def _agree():
    import torch
    return binding._torch_stream(None) == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("where", ["default", "side", "nested", "thread"])
def test_current_stream_is_torchs(where):
    import torch
    torch.empty(1, device="cuda:0")
    if where == "default":
        assert _agree()
        return
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        assert _agree() and binding._torch_stream(None) == a.cuda_stream
        if where == "nested":
            with torch.cuda.stream(b):
                assert _agree() and binding._torch_stream(None) == b.cuda_stream
        if where == "thread":
            got = []
            t = threading.Thread(target=lambda: got.append((_agree(), binding._torch_stream(None))))
            t.start()
            t.join()
            assert got == [(True, torch.cuda.default_stream().cuda_stream)]
        assert binding._torch_stream(None) == a.cuda_stream
    assert _agree()
