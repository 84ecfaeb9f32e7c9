"""Scratch that the binding allocates for a call belongs to the call's stream
(no GPU: the library, the allocator and the streams are stand-ins)."""
import contextlib
import types

import pytest
import torch

from paper_2512_20943_amd import gs


@pytest.mark.parametrize("call", ["usage", "cull"])
@pytest.mark.parametrize("given", [True, False])
def test_scratch_is_allocated_on_the_calls_stream(monkeypatch, call, given):
    entered, seen = [], []

    @contextlib.contextmanager
    def on(stream):
        entered.append(stream)
        yield
        entered.pop()

    plain = torch.empty

    def empty(*size, **kw):
        seen.append(entered[-1] if entered else None)
        return plain(*size, **kw)

    lib = types.SimpleNamespace(
        gs_usage_masks_workspace_size=lambda n: 64, gs_cull_workspace_size=lambda n: 64,
        gs_usage_masks=lambda *a: 0, gs_cull_low_opacity=lambda *a: 0)
    ctx = types.SimpleNamespace(lib=lib, handle=None, check=lambda st: None)
    monkeypatch.setattr(gs, "load", lambda: lib)
    monkeypatch.setattr(gs, "_stream", lambda s: None)
    monkeypatch.setattr(gs, "_ptr", lambda t: None)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch, "empty", empty)
    side = object() if given else None
    x = torch.zeros(16)
    if call == "usage":
        gs.gs_usage_masks(ctx, x.int(), 16, 4, 4, [3], x.byte(), stream=side)
    else:
        gs.gs_cull_low_opacity(ctx, x, 16, 0.5, x.int(), stream=side)
    assert seen == [side]
