"""A forked child must not use its parent's GPU: the binding asks torch for the stream again, which
refuses there.  (The stream handle is kept after the first call.)"""
import os

import paper_2604_06664_amd as fdy


def test_a_forked_child_asks_for_its_stream_again(monkeypatch):
    monkeypatch.setattr(fdy, "_raw_stream", lambda: 7)  # as after a first call
    assert fdy._stream(None) == 7
    pid = os.fork()
    if pid == 0:
        os._exit(0 if fdy._raw_stream is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert fdy._stream(None) == 7
