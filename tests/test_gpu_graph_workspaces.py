"""Graphs and workspaces: replays of a captured train step stay right whatever
calls come between them (predictions of more rows than the batch, a larger
train step, which replaces the workspaces, new allocations); predictions can be
captured after training with smaller batches, since they allocate nothing."""
import ctypes

import numpy as np
import pytest
import torch

from tests.test_gpu_surrogate import DEV, padded_from, problem

pytestmark = pytest.mark.gpu


class Blocks:
    """Device blocks of their own (not from torch's pool) holding a pattern."""

    def __init__(self, sizes):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.blocks = []
        for n in sizes:
            p = ctypes.c_void_p()
            assert self.hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(n)) == 0
            assert self.hip.hipMemset(p, 0x5A, ctypes.c_size_t(n)) == 0
            self.blocks.append((p, n))
        torch.cuda.synchronize()

    def untouched_then_free(self):
        torch.cuda.synchronize()
        ok = True
        for p, n in self.blocks:
            buf = (ctypes.c_ubyte * n)()
            assert self.hip.hipMemcpy(buf, p, ctypes.c_size_t(n), 2) == 0       # device to host
            ok = ok and bool((np.frombuffer(buf, np.uint8) == 0x5A).all())
            assert self.hip.hipFree(p) == 0
        return ok


SIZES = [1 << k for k in range(12, 22)] * 2      # 4 KB to 2 MB: the sizes of these nets' workspaces


@pytest.mark.parametrize("widths,bf16", [((6, 64, 64, 256), False), ((6, 100, 77, 1001), False),
                                         ((6, 64, 64, 256), True)])
def test_replays_survive_predictions_and_larger_steps(widths, bf16):
    """Replays with predictions of more rows than the batch, new allocations and a
    larger eager step between them equal the same calls made eagerly, bit for
    bit, and the new allocations keep their contents."""
    from paper_2309_16743_amd import OT_BF16, OT_FP32, Surrogate
    B, big = 32, 70
    _, X, U = problem(widths, big, seed=3)
    x, u = padded_from(X[:B]), padded_from(U[:B])
    xl, ul = padded_from(X), padded_from(U)
    xp = padded_from(problem(widths, 300, seed=4)[1])
    out = {}
    for graph in (False, True):
        s = Surrogate(widths, precision=OT_BF16 if bf16 else OT_FP32, seed=5, max_batch=B)
        y = [padded_from(np.zeros((n, widths[-1]), np.float32)) for n in (80, 300, 256)]
        losses = torch.zeros(6, device=DEV)
        loss = torch.zeros(1, device=DEV)
        s.train_step(x, u, loss=losses[0:1])
        torch.cuda.synchronize()
        s.set_device_step(True)
        g = None
        if graph:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                s.train_step(x, u, loss=loss)

        def step(i):
            if g is None:
                s.train_step(x, u, loss=losses[i:i + 1])
            else:
                g.replay()
                losses[i].copy_(loss[0])
        step(1)
        s.predict(xp[:80], y[0])
        blocks = Blocks(SIZES)
        step(2)
        s.predict(xp, y[1])
        step(3)
        s.train_step(xl, ul, loss=losses[4:5])          # replaces the workspaces
        more = Blocks(SIZES)
        step(5)
        s.predict(xp[:256], y[2])
        assert blocks.untouched_then_free() and more.untouched_then_free()
        s.set_device_step(False)
        state = [s.get_adam_state(l) for l in range(len(widths) - 1)]
        assert state[0][2] == 6
        out[graph] = ([losses.cpu().numpy()] + [t.cpu().numpy() for t in y] +
                      [a for l in range(len(widths) - 1) for a in s.get_params(l)] +
                      [a for m, v, _ in state for a in (*m, *v)])
        s.close()
    assert all(np.isfinite(a).all() for a in out[False])
    assert all(np.array_equal(a, b) for a, b in zip(out[False], out[True]))


@pytest.mark.parametrize("widths,bf16", [((6, 64, 64, 256), False), ((6, 300, 200, 5000), False),
                                         ((6, 96, 160, 61450), True)])
def test_prediction_captured_after_small_batches(widths, bf16):
    """A prediction of more rows than any batch so far can be captured (nothing
    is allocated), and every replay equals the eager call."""
    from paper_2309_16743_amd import OT_BF16, OT_FP32, Surrogate
    _, X, U = problem(widths, 8, seed=6)
    s = Surrogate(widths, precision=OT_BF16 if bf16 else OT_FP32, seed=7, max_batch=8)
    x, u = padded_from(X), padded_from(U)
    s.train_step(x, u)
    torch.cuda.synchronize()
    for n in (40, 200, 300):
        xp = padded_from(problem(widths, n, seed=n)[1])
        y = padded_from(np.zeros((n, widths[-1]), np.float32))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            s.predict(xp, y)
        ref = padded_from(np.zeros((n, widths[-1]), np.float32))
        for _ in range(2):
            y.zero_()
            g.replay()
            s.predict(xp, ref)
            torch.cuda.synchronize()
            assert torch.equal(y, ref)
            s.train_step(x, u)                          # the next replay predicts with new weights
    s.close()
