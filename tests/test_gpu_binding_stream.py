"""The binding's launches go to the stream that torch calls current, in and out of a stream context and in other threads."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_stream_is_torchs_current_stream():
    import torch
    from paper_2410_21271_amd import binding
    torch.zeros(1, device="cuda")
    seen = []

    def same():
        seen.append(int(binding._stream()) == torch.cuda.current_stream().cuda_stream)

    same()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        same()
        seen.append(int(binding._stream()) == side.cuda_stream)
        t = threading.Thread(target=same)                 # a thread starts on its own default stream
        t.start()
        t.join()
    same()
    assert seen and all(seen)


def test_missing_pointers_are_refused():
    import paper_2410_21271_amd as eora
    with pytest.raises(eora.EoraError) as e:
        eora.linear_q(None, None, None, None, None, None, None, None, None, 1, 128, 16, 0, 4, 128, 16, None)
    assert e.value.status == -1
