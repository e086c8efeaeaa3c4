"""The stream that the binding passes on when none is given: torch's current one, on every thread."""
import threading

import pytest
import torch

from paper_2506_12024_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["default", "side", "external"])
def test_the_current_stream_is_passed_on(kind):
    side = torch.cuda.Stream() if kind != "default" else torch.cuda.default_stream()
    if kind == "external":
        side = torch.cuda.ExternalStream(side.cuda_stream)
    seen = {}

    def other():
        seen["thread"] = binding._stream(None)  # a thread of its own starts on the default stream

    with torch.cuda.stream(side):
        assert binding._stream(None) == torch.cuda.current_stream().cuda_stream == side.cuda_stream
        t = threading.Thread(target=other)
        t.start()
        t.join()
    assert seen["thread"] == torch.cuda.default_stream().cuda_stream
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream
    assert binding._stream(side) == side.cuda_stream and binding._stream(7) == 7
