"""Scratch that the tensor functions allocate for one call belongs to the stream the call is enqueued on.  It is freed when the function
returns, before the call has run, so on any other stream its memory could be given away while the call still uses it.  Runs without a
GPU: the library's entry points are recorded in place of being called."""
import contextlib
import types

import pytest
import torch

from paper_2512_21450_amd import binding as B


class OnDevice(torch.Tensor):
    is_cuda = property(lambda self: True)


def tensor(*shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype).as_subclass(OnDevice)


def decode(dtype, d, **kw):
    t = lambda *s: tensor(*s, dtype=dtype)
    n = lambda k: torch.zeros(k, dtype=torch.int32)
    return B.rl_decode_attn(t(2, 1, d), t(2, 1, 800, d), t(2, 1, 800, d), n(2), t(2, 1, 40, d), t(2, 1, 40, d), n(2), 0.1, 1, **kw)


def paged(dtype, d, **kw):
    t = lambda *s: tensor(*s, dtype=dtype)
    n = lambda *k: torch.zeros(k, dtype=torch.int32)
    return B.rl_decode_attn_paged(t(2, 1, d), t(2, 1, 800, d), t(2, 1, 800, d), n(2), t(4, 1, 32, d), t(4, 1, 32, d), n(2, 2), n(2), 0.1, 1, **kw)


def tree(**kw):
    t = lambda *s: tensor(*s, dtype=torch.bfloat16)
    n = lambda k: torch.zeros(k, dtype=torch.int32)
    return B.rl_decode_attn_tree(t(2, 1, 128), [(t(1, 1, 64, 128), t(1, 1, 64, 128), n(1), 2)], t(2, 1, 8, 128), t(2, 1, 8, 128), n(2), 0.1, **kw)


CALLS = {"rl_decode_attn": [lambda **kw: decode(torch.float32, 64, **kw), lambda **kw: decode(torch.bfloat16, 128, **kw)],
         "rl_decode_attn_paged": [lambda **kw: paged(torch.float32, 64, **kw), lambda **kw: paged(torch.bfloat16, 128, **kw)],
         "rl_decode_attn_tree": [tree],
         "rl_token_logprob": [lambda **kw: B.rl_token_logprob(tensor(4, 32000), torch.zeros(4, dtype=torch.int32), **kw)],
         "rl_policy_loss": [lambda **kw: B.rl_policy_loss(tensor(4, 8), tensor(4, 8), tensor(4), torch.zeros(4, dtype=torch.int32), 0.2, 0.2, **kw)]}


@pytest.mark.parametrize("name,k", [(n, k) for n, c in CALLS.items() for k in range(len(c))])
def test_scratch_is_allocated_on_the_stream_of_the_call(name, k, monkeypatch):
    on, taken, seen = [], {}, []

    @contextlib.contextmanager
    def stream_context(s):
        on.append(s)
        yield
        on.pop()

    empty = torch.empty

    def recorded_empty(*a, **kw):
        t = empty(*a, **kw)
        if kw.get("dtype") == torch.uint8:
            taken[t.data_ptr()] = on[-1] if on else None
        return t

    def entry(desc, handle, *_):
        ds = desc._obj
        seen.append((ds.workspace, ds.workspace_bytes, handle))
        return 0

    class Stream:
        def __init__(self, cuda_stream):
            self.cuda_stream = cuda_stream

    monkeypatch.setattr(torch.cuda, "stream", stream_context)
    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device: Stream(handle))
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device: Stream(0))
    monkeypatch.setattr(torch, "empty", recorded_empty)
    monkeypatch.setattr(B._lib, name, entry)
    monkeypatch.setattr(B, "_stream_handle", lambda stream, like: 0 if stream is None else stream.cuda_stream)
    for stream in (None, Stream(77), types.SimpleNamespace(cuda_stream=78), types.SimpleNamespace(cuda_stream=0)):
        CALLS[name][k](stream=stream)
        ws, nbytes, handle = seen[-1]
        assert nbytes > 0 and handle == (0 if stream is None else stream.cuda_stream)
        assert taken[ws] is None if stream is None else taken[ws].cuda_stream == stream.cuda_stream
