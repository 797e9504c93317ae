"""The binding's stream handle and device guard are those of torch's public
interface, and calls run on the stream that is current."""
import pytest
import torch

from paper_2607_22586_amd import binding as bd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("guard", [bd._RawGuard, torch.cuda.device])
@pytest.mark.parametrize("handle", [bd._raw_stream, bd._public_stream])
def test_calls_run_on_the_current_stream(monkeypatch, guard, handle):
    monkeypatch.setattr(bd, "_on", guard)
    monkeypatch.setattr(bd, "_raw_stream", handle)
    dev, side = torch.device("cuda:0"), torch.cuda.Stream("cuda:0")
    assert bd._stream(dev) == torch.cuda.current_stream(dev).cuda_stream
    with torch.cuda.stream(side):
        assert bd._stream(dev) == side.cuda_stream
        with bd._on(dev):
            assert torch.cuda.current_device() == 0 and bd._stream(dev) == side.cuda_stream
        score = bd.shape_scores(None, bd.MMSKV_SHAPE_STREAMING, 1, 2, 1000, sinks=4, device=dev)
        last = score[..., -1].sum()              # ordered behind the call on that stream
    side.synchronize()
    assert float(last) == 2 * 999
