"""Calls without a stream go to torch's current one, whichever that is and in whichever thread."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_default_stream_of_a_call_is_the_current_one():
    from paper_2507_17307_amd import binding as B
    torch.zeros(1, device="cuda")
    side, seen = torch.cuda.Stream(), []

    def note():
        seen.append((B._stream(None), torch.cuda.current_stream().cuda_stream))

    note()
    with torch.cuda.stream(side):
        note()
        t = threading.Thread(target=note)                    # a thread of its own starts on the default stream
        t.start()
        t.join()
    note()
    assert len(seen) == 4                                    # (an exception in the thread leaves three)
    assert all(a == b for a, b in seen) and seen[1][0] == side.cuda_stream != seen[2][0], seen
