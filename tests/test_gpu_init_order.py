"""A workspace that the caller's stream is still writing when the context is made:
the uploads come after what was queued.  (The order of the calls themselves is
tested on the CPU.)"""
import numpy as np
import pytest
import torch

import swf_workloads as W

pytestmark = pytest.mark.gpu


def test_pending_work_on_the_workspace(monkeypatch):
    from paper_2512_16889_amd import swf as S
    prob = W.config_2d(n=64, L=160.0, dt=0.05, t_half=0.5, n_solves=2)
    with S.Context(prob, precision="fp64") as ctx:
        ctx.step()
        ref = [ctx.get_psi(i) for i in range(2)]
    real = torch.empty
    load = torch.full((1 << 28,), 1.0, device="cuda")     # 1 GiB: its passes keep the stream busy for milliseconds

    def busy(*a, **k):
        ws = real(*a, **k)
        for _ in range(20):
            load.mul_(1.0)
        ws.fill_(0xFF)
        return ws
    with monkeypatch.context() as m:
        m.setattr(S.torch, "empty", busy)
        ctx = S.Context(prob, precision="fp64")
    with ctx:
        ctx.step()
        for i in range(2):
            assert np.array_equal(ctx.get_psi(i), ref[i])
