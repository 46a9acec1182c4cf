"""The partial sums of every Gram fit the buffer they are given (CPU only).

tests/host_gram_room.cpp is the library's host code compiled without its
kernels: each launch of a block's or a closing QR's Gram is recorded instead of
made, over block widths 1..128, real and complex, both data types and heights
up to 2^20, and the last double written is compared with the end of the buffer
that the workspace carve holds for it.  Blocks of 65 to 128 columns write up to
63 partials of their full square and the sum behind them, which from about a
thousand rows on is more than the partials of the narrower blocks take.
"""
from host_cc import run_host


def test_gram_partials_fit_their_buffers(tmp_path):
    run = run_host("host_gram_room.cpp", tmp_path)
    assert run.returncode == 0, run.stdout[-2000:]
    assert " 0 overrun" in run.stdout
