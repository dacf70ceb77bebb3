"""The served pipeline's limit of 4096 launches counts phase steps, whatever the
batched form makes of them (host checks only, no device)."""
import ctypes

import pytest

from paper_1804_03787_amd import msgpm
from tests.test_host_failures import _err, _lib, _server, _submit


# features, initial state (2), half-sweeps, final refresh and output, filling and its clear; per level
# two stages of four steps, check (2), cue 2 (4), update, lists (3), half-sweeps of two kinds of pixels
@pytest.mark.parametrize("kw,rest", [
    (dict(blocks=(), iters=8), 1 + 2 + 16 + 2 + 1),
    (dict(blocks=(), iters=0), 1 + 2 + 1 + 2 + 1),
    (dict(blocks=(32, 16), iters=5), 1 + 2 + 10 + 2 + 1 + 2 * (8 + 2 + 1 + 3 + 20)),
    (dict(blocks=(16,), iters=0, histeq=True, cue_unique=True), 3 + 1 + 2 + 1 + 2 + 1 + 8 + 2 + 4 + 1 + 3 + 2),
])
def test_launch_limit_counts_phase_steps(kw, rest):
    h = _server(1 << 40)
    ok = msgpm.make_params(64, 48, fill_sweeps=4096 - rest, **kw)
    st, ticket = _submit(h, ok)
    assert st == 0, _err()
    assert _lib().msgpm_server_cancel(h, ticket, ctypes.byref(ctypes.c_int())) == 0
    st, _ = _submit(h, msgpm.make_params(64, 48, fill_sweeps=4097 - rest, **kw))
    assert st == msgpm.E_UNSUPPORTED and "4096 launches" in _err()
    assert _lib().msgpm_server_destroy(h) == 0
