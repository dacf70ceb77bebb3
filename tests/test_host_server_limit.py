"""The served pipeline's limit of 4096 launches does not count the moment
launches of its PatchMatch passes (host checks only, no device)."""
import ctypes

from paper_1804_03787_amd import msgpm
from tests.test_host_failures import _err, _lib, _server, _submit


def test_launch_limit_counts_what_it_counted_before_the_moments():
    # features, initial state (2), 16 half-sweeps, final refresh and output, filling and its clear
    rest = 1 + 2 + 16 + 2 + 1
    h = _server(1 << 40)
    ok = msgpm.make_params(64, 48, blocks=(), iters=8, fill_sweeps=4096 - rest)
    st, ticket = _submit(h, ok)
    assert st == 0, _err()
    assert _lib().msgpm_server_cancel(h, ticket, ctypes.byref(ctypes.c_int())) == 0
    st, _ = _submit(h, msgpm.make_params(64, 48, blocks=(), iters=8, fill_sweeps=4097 - rest))
    assert st == msgpm.E_UNSUPPORTED and "4096 launches" in _err()
    assert _lib().msgpm_server_destroy(h) == 0
