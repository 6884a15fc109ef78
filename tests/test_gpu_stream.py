"""Calls go to the stream that is current when they are made, bound calls too."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    from paper_2507_00715_amd import binding as B
    side, main = torch.cuda.Stream(), torch.cuda.current_stream()
    assert B._stream() == main.cuda_stream
    with torch.cuda.stream(side):
        assert B._stream() == side.cuda_stream
        with torch.cuda.stream(main):
            assert B._stream() == main.cuda_stream
    assert B._stream() == main.cuda_stream
    cu, q_pos, gen_len = (torch.tensor(x, dtype=torch.int32, device="cuda:0") for x in ([0, 5, 9], [0, 0], [0, 0]))
    call = B.bind_decode_step_positions(cu, None, 2, 2, 3, q_pos, gen_len)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)           # the side stream is busy: what the call writes is not there yet ...
        call()
        done = torch.cuda.Event()
        done.record(side)
    assert not done.query()
    main.wait_event(done)                       # ... and is once the side stream has been waited for
    assert q_pos.tolist() == [8, 7] and gen_len.tolist() == [3, 3]
