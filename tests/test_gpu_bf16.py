"""Mixed-precision (bf16 operands, fp32 accumulation / master weights / Adam)
surrogate against the oracle's bf16 mode, which rounds exactly the operands the
GPU rounds (activations of layers >= 2, the weight copy, dY and every dZ) and
accumulates in fp64.  Tolerance: 2e-2 relative L2 per tensor, and for
gradients also element-wise (every entry within 2e-2 of the tensor's largest).
The two 1000x1000 nets are checked at their full 10^6-wide output layer."""
import numpy as np
import pytest
import torch

from fixtures import configs, heat
from oracle import mlp, runner

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = 2e-2


def rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def close(a, b, tol):
    """Relative L2 within tol and every element within tol of the largest
    reference entry (so that one wrong output unit among thousands fails)."""
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    scale = max(float(np.max(np.abs(b))), 1e-30)
    return rel(a, b) < tol and float(np.max(np.abs(a - b))) / scale < tol


def padded_from(arr):
    rows, d = arr.shape
    ld = (d + 7) // 8 * 8
    t = torch.zeros(rows, ld, device=DEV)[:, :d]
    t.copy_(torch.from_numpy(np.ascontiguousarray(arr, dtype=np.float32)))
    return t


def problem(widths, B, seed):
    rng = np.random.default_rng(seed)
    params = []
    for l in range(len(widths) - 1):
        fi, fo = widths[l], widths[l + 1]
        bound = 1 / np.sqrt(fi)
        params.append((rng.uniform(-bound, bound, (fo, fi)).astype(np.float32).astype(np.float64),
                       rng.uniform(-bound, bound, fo).astype(np.float32).astype(np.float64)))
    X = np.concatenate([rng.uniform(100, 500, (B, 5)), rng.uniform(0.01, 1.0, (B, 1))], axis=1)
    U = rng.uniform(100, 500, (B, widths[-1]))
    return params, X.astype(np.float32), U.astype(np.float32)


def make_gpu(widths, params, B, flags=0):
    from paper_2309_16743_amd import OT_BF16, Surrogate
    s = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=0, flags=flags)
    for l, (W, b) in enumerate(params):
        s.set_params(l, W.astype(np.float32), b.astype(np.float32))
    return s


SHAPES = [
    ((6, 64, 64, 256), 32),
    ((6, 100, 77, 1001), 50),          # ragged widths, 64 x 64 tiles, partial tiles
    ((6, 256, 256, 4000), 128),        # split-K input gradient
    ((6, 128, 128, 128, 300), 64),     # three hidden layers
    ((6, 512, 512, 20000), 512),       # pipelined 256 x 128 kernel, the bf16 workloads' batch
    ((6, 512, 512, 30001), 320),       # pipelined kernel with ragged M and N (clamped edges)
    ((6, 1024, 1024, 69984), 512),     # ping-pong forward, ragged N; split-K input gradient (63 splits, ragged last split)
    ((6, 512, 512, 69984), 300),       # ping-pong forward and split-K input gradient with a ragged batch (M = 300)
    ((6, 2048, 2048, 2048, 4096), 1024),   # the deep 1000x1000 net's hidden widths and batch
    ((6, 16, 16, 1), 1),               # one sample, one output
    ((6, 40, 24, 9), 3),               # three samples, ragged narrow widths
    ((6, 64, 83, 500), 36),            # fused update whose last column group is partial and starts a 16-column fragment
    ((6, 64, 470, 30001), 64),         # the same on the pipelined kernel's tiles
    ((6, 96, 160, 61450), 100),        # up to 128 rows: 128 x 256 forward and input gradient, k padded from 61450
    ((6, 64, 256, 61440), 129),        # just above: 256 x 256 forward (half its rows clamped) and input gradient
    ((6, 96, 128, 15361), 64),         # up to 64 rows: 64 x 64 forward
    ((6, 512, 512, 19600), 512),       # 256 x 128 input gradient in short splits, k padded from 19600
]


@pytest.mark.parametrize("widths,B", SHAPES)
def test_one_train_step_bf16(widths, B):
    """Kept gradients: loss, every gradient and every parameter after Adam
    against the oracle.  Fused output-layer Adam (the default): every
    parameter against the oracle, and against the kept-gradient step within
    1e-5 (the fused GEMM never splits k, the stored one may, so the gradient
    sums can differ in rounding order)."""
    from paper_2309_16743_amd import OT_SURROGATE_KEEP_GRADS
    print(f"bf16 one train step widths={widths} B={B}", flush=True)
    params, X, U = problem(widths, B, seed=sum(widths) + B)
    s = make_gpu(widths, params, B, flags=OT_SURROGATE_KEEP_GRADS)
    f = make_gpu(widths, params, B)
    Xd, Ud = padded_from(X), padded_from(U)
    loss, loss_f = torch.zeros(1, device=DEV), torch.zeros(1, device=DEV)
    s.train_step(Xd, Ud, loss=loss)
    f.train_step(Xd, Ud, loss=loss_f)
    torch.cuda.synchronize()
    o_loss, o_grads = mlp.loss_and_grads(params, X.astype(np.float64), U.astype(np.float64), bf16=True)
    o_new = mlp.Adam(lr=1e-3).step(params, o_grads)
    assert abs(loss.item() - o_loss) / o_loss < 1e-3
    assert loss_f.item() == loss.item()
    for l in range(len(widths) - 1):
        gW, gb = s.get_grads(l)
        assert close(gW, o_grads[l][0], TOL), (l, rel(gW, o_grads[l][0]))
        assert close(gb, o_grads[l][1], TOL), (l, rel(gb, o_grads[l][1]))
        W, b = s.get_params(l)
        assert rel(W, o_new[l][0]) < TOL and rel(b, o_new[l][1]) < TOL
        Wf, bf = f.get_params(l)
        assert rel(Wf, o_new[l][0]) < TOL and rel(bf, o_new[l][1]) < TOL
        assert rel(Wf, W) < 1e-5 and rel(bf, b) < 1e-5, (l, rel(Wf, W))
    s.close()
    f.close()


@pytest.mark.parametrize("widths,n", [((6, 64, 64, 256), 40), ((6, 100, 77, 1001), 77), ((6, 64, 96, 61441), 1),
                                      ((6, 64, 96, 61443), 128), ((6, 64, 96, 61447), 200),
                                      ((6, 64, 96, 999), 300)])   # 300 rows: two passes
def test_predict_bf16(widths, n):
    params, X, _ = problem(widths, n, seed=5)
    s = make_gpu(widths, params, 32)
    Y = padded_from(np.zeros((n, widths[-1]), np.float32))
    s.predict(padded_from(X), Y)
    torch.cuda.synchronize()
    assert rel(Y.cpu().numpy(), mlp.predict(params, X.astype(np.float64), bf16=True)) < 1e-3
    s.close()


def test_tiny_workload_100_steps_bf16():
    from paper_2309_16743_amd import OT_BF16
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    ref = runner.run(w, inputs, fields, n_steps=100, bf16=True)
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, precision=OT_BF16, lr=w.lr, record_steps=100)
    tr.run(100)
    torch.cuda.synchronize()
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < TOL
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < TOL and rel(b, ref["params"][l][1]) < TOL
    tr.close()


def full_width_step(widths, B, seed, chunk, fp64_report=False):
    """One bf16 train step of a net whose output layer is 10^6 wide, against
    the oracle computed by output-column chunks (oracle.mlp
    output_layer_by_columns, then hidden_grads for the layers below).

    Inputs: hidden layers, X and the output bias from numpy's seeded
    generator; W_L (10^6 x H) and the targets U (B x 10^6) from torch's
    seeded generator on the device (too large for a host generator in a test
    budget), copied to host memory for the oracle and uploaded to the
    library through surrogate_set_params.  W_L is drawn bf16-representable,
    so the oracle skips its (identity) weight rounding at this size.

    Checks: loss; every gradient of the hidden layers (relative L2 and
    element-wise, 2e-2); the output bias gradient over all 10^6 units; the
    output weight-gradient rows and updated rows at sampled units; the fused
    step's parameters bit-identical to the kept-gradient step's."""
    import time
    from paper_2309_16743_amd import OT_BF16, OT_SURROGATE_KEEP_GRADS, Surrogate
    t0 = time.perf_counter()
    L, D, H = len(widths) - 1, widths[-1], widths[-2]
    rng = np.random.default_rng(seed)
    hidden = []
    for l in range(L - 1):
        bound = 1 / np.sqrt(widths[l])
        hidden.append((rng.uniform(-bound, bound, (widths[l + 1], widths[l])).astype(np.float32).astype(np.float64),
                       rng.uniform(-bound, bound, widths[l + 1]).astype(np.float32).astype(np.float64)))
    bL = rng.uniform(-1 / np.sqrt(H), 1 / np.sqrt(H), D).astype(np.float32)
    X = np.concatenate([rng.uniform(100, 500, (B, 5)), rng.uniform(0.01, 1.0, (B, 1))], axis=1).astype(np.float32)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    W_dev = torch.empty(D, H, device=DEV).uniform_(-1 / np.sqrt(H), 1 / np.sqrt(H), generator=g)
    W_dev.view(torch.int32).bitwise_and_(-65536)            # bf16-representable values
    U_dev = torch.empty(B, D, device=DEV).uniform_(100, 500, generator=g)
    W_host = W_dev.cpu().numpy()
    del W_dev
    assert not np.any(W_host.view(np.uint32) & np.uint32(0xFFFF))
    s = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=0, flags=OT_SURROGATE_KEEP_GRADS)
    f = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=0)       # fused output-layer Adam
    for sur in (s, f):
        for l, (W, b) in enumerate(hidden):
            sur.set_params(l, W.astype(np.float32), b.astype(np.float32))
        sur.set_params(L - 1, W_host, bL)
    Xd = padded_from(X)
    loss = torch.zeros(1, device=DEV)
    s.train_step(Xd, U_dev, loss=loss)
    f.train_step(Xd, U_dev)
    torch.cuda.synchronize()
    U_host = U_dev.cpu().numpy()
    del U_dev
    print(f"  inputs and GPU steps: {time.perf_counter() - t0:.1f} s", flush=True)
    # the oracle, by column chunks of the output layer
    js = np.array([0, 1, 777, 123457, 500000, 999999])
    X64 = X.astype(np.float64)

    def oracle(bf16):
        Zs, As, Zh = mlp.forward(hidden, X64, bf16=bf16)
        rounded = (mlp.BF16_ROUNDED - {"weight"}) if bf16 else None
        o_loss, dA, db, dWj = mlp.output_layer_by_columns(np.maximum(Zh, 0.0), lambda a, c: W_host[a:c], bL,
                                                          lambda a, c: U_host[:, a:c], D, chunk, bf16=bf16,
                                                          rows=js, rounded=rounded)
        return o_loss, mlp.hidden_grads(hidden, Zs, dA, As, bf16=bf16), db, dWj

    o_loss, o_hidden, o_db, o_dWj = oracle(True)
    print(f"  oracle: {time.perf_counter() - t0:.1f} s", flush=True)
    assert abs(loss.item() - o_loss) / o_loss < TOL, (loss.item(), o_loss)
    for l in range(L - 1):
        gW, gb = s.get_grads(l)
        assert close(gW, o_hidden[l][0], TOL), (l, rel(gW, o_hidden[l][0]))
        assert close(gb, o_hidden[l][1], TOL), (l, rel(gb, o_hidden[l][1]))
    gW, gb = s.get_grads(L - 1)
    assert close(gb, o_db, TOL), rel(gb, o_db)
    assert close(gW[js], o_dWj, TOL), rel(gW[js], o_dWj)
    del gW
    Wj = W_host[js].astype(np.float64)
    newWj = mlp.Adam(lr=1e-3).step([(Wj, bL[js].astype(np.float64))], [(o_dWj, o_db[js])])[0][0]
    W, b = s.get_params(L - 1)
    assert rel(W[js], newWj) < TOL
    Wf, bf = f.get_params(L - 1)
    # the weight gradient is not split over k on either path: same sums, same Adam
    assert np.array_equal(Wf, W) and np.array_equal(bf, b)
    del W, Wf
    print(f"  loss {loss.item():.6g} (oracle {o_loss:.6g}); checks done at {time.perf_counter() - t0:.1f} s",
          flush=True)
    if fp64_report:
        p_loss, p_hidden, p_db, _ = oracle(False)
        r = [abs(loss.item() - p_loss) / p_loss] + [rel(s.get_grads(l)[0], p_hidden[l][0]) for l in range(L - 1)]
        print("  bf16 path against the pure fp64 oracle (loss, hidden dW): " + ", ".join(f"{x:.2e}" for x in r),
              flush=True)
        assert max(r) < 5e-2
    s.close()
    f.close()


def test_full_width_step_bf16():
    """6-1024-1024-1,000,000 at batch 512 (the 1000x1000 workload's net)."""
    print("full-width bf16 step 6-1024-1024-1e6, B 512", flush=True)
    full_width_step((6, 1024, 1024, 1_000_000), 512, seed=5, chunk=32768, fp64_report=True)


def test_full_width_step_deep_bf16():
    """6-2048-2048-2048-1,000,000 at batch 1024 (the deep 1000x1000 workload's net)."""
    print("full-width bf16 step 6-2048-2048-2048-1e6, B 1024", flush=True)
    full_width_step((6, 2048, 2048, 2048, 1_000_000), 1024, seed=8, chunk=16384)


def test_full_width_targets_in_place_bf16():
    """6-1024-1024-1,000,000 at batch 512 with the targets read in place from
    a 600-row array through row indices (the benchmark's path): the same loss
    and the same parameters, bit for bit, as the step on the gathered rows."""
    from paper_2309_16743_amd import OT_BF16, Surrogate
    widths, B, seed, n_rows = (6, 1024, 1024, 1_000_000), 512, 5, 600
    rng = np.random.default_rng(12)
    X = np.concatenate([rng.uniform(100, 500, (B, 5)), rng.uniform(0.01, 1.0, (B, 1))], axis=1).astype(np.float32)
    slab = torch.empty(n_rows, widths[-1], device=DEV)
    slab.uniform_(100, 500, generator=torch.Generator(device=DEV).manual_seed(3))
    rows = torch.from_numpy(rng.integers(0, n_rows, B).astype(np.int32)).to(DEV)
    a = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=seed)
    g = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=seed)
    Xd = padded_from(X)
    la, lg = torch.zeros(1, device=DEV), torch.zeros(1, device=DEV)
    a.train_step_rows(Xd, slab.data_ptr(), widths[-1], rows, n_rows, loss=la)
    gathered = slab[rows.long()]
    g.train_step(Xd, gathered, loss=lg)
    torch.cuda.synchronize()
    del gathered
    assert la.item() == lg.item()
    for l in range(3):
        Wa, ba = a.get_params(l)
        Wg, bg = g.get_params(l)
        assert np.array_equal(Wa, Wg) and np.array_equal(ba, bg), l
    a.close()
    g.close()


def test_mid_size_online_schedule_bf16():
    """A 6-512-512-19,600 bf16 net (140x140 heat fields) at batch 512 through
    the online loop as the benchmark runs it (two streams, targets read in
    place, pipelined GEMM kernels, output-layer Adam fused into its weight
    gradient), with a 700-slot reservoir so that puts evict during the run:
    10 steps, slots bit-exact, loss series and final parameters within 2e-2
    relative L2 of the oracle's bf16 mode."""
    import dataclasses
    from paper_2309_16743_amd import OT_BF16
    from paper_2309_16743_amd.online import OnlineTrainer
    w = dataclasses.replace(configs.HEAT100, grid=140, n_sims=24, wave=24, widths=(6, 512, 512, 19600),
                            precision="bf16", batch=512, capacity=700, threshold=512)
    print(f"bf16 mid-size online schedule widths={w.widths} B={w.batch} C={w.capacity}", flush=True)
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    n = 10
    ref = runner.run(w, inputs, fields, n_steps=n)
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, precision=OT_BF16, lr=w.lr, record_steps=n, overlap=True)
    tr.run(n)
    torch.cuda.synchronize()
    assert tr.res.stats()["total_evicted"] > 0
    slots = tr.slot_log.cpu().numpy()
    for i in range(n):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < TOL
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < TOL and rel(b, ref["params"][l][1]) < TOL
    tr.close()


def test_fused_steps_predict_and_restart_bf16():
    """Five fused bf16 steps (the output layer's Adam in its weight-gradient
    epilogue) against the oracle's five: the loss of every step and the final
    parameters; predictions after an odd and an even number of steps; a
    checkpoint taken after step 3, restored into a fresh surrogate, continues
    bit for bit through steps 4 and 5."""
    from paper_2309_16743_amd import OT_BF16, Surrogate
    widths, B = (6, 512, 512, 20000), 512
    params, X, U = problem(widths, B, seed=77)
    f = make_gpu(widths, params, B)
    Xd, Ud = padded_from(X), padded_from(U)
    o_params = params
    opt = mlp.Adam(lr=1e-3)
    Xq = X[:64].astype(np.float64)
    for step in range(5):
        loss = torch.zeros(1, device=DEV)
        f.train_step(Xd, Ud, loss=loss)
        o_loss, o_grads = mlp.loss_and_grads(o_params, X.astype(np.float64), U.astype(np.float64), bf16=True)
        o_params = opt.step(o_params, o_grads)
        torch.cuda.synchronize()
        assert abs(loss.item() - o_loss) / o_loss < 1e-3, (step, loss.item(), o_loss)
        if step in (2, 3):
            Y = padded_from(np.zeros((64, widths[-1]), np.float32))
            f.predict(padded_from(X[:64]), Y)
            torch.cuda.synchronize()
            assert rel(Y.cpu().numpy(), mlp.predict(o_params, Xq, bf16=True)) < 1e-3, step
        if step == 2:
            blob = f.checkpoint()
    for l in range(3):
        W, b = f.get_params(l)
        assert rel(W, o_params[l][0]) < TOL and rel(b, o_params[l][1]) < TOL, l
    # restart from the checkpoint taken after step 3 and take steps 4 and 5 again
    g = Surrogate(widths, precision=OT_BF16, max_batch=B, seed=123)
    g.restore(blob)
    for _ in range(2):
        g.train_step(Xd, Ud)
    torch.cuda.synchronize()
    for l in range(3):
        for a, c in zip(f.get_params(l), g.get_params(l)):
            assert np.array_equal(a, c), l
    f.close()
    g.close()


@pytest.mark.parametrize("widths,B,i", [((6, 16, 16, 40), 1, 4), ((6, 64, 96, 61450), 100, 50)])
def test_infinite_output_bias_stays_in_its_products(widths, B, i):
    """dY's rows are padded with zeros to whole k tiles of the input gradient;
    the weight rows that meet the padding are zero whatever the parameters that
    follow W_L hold.  One infinite bias makes its column of dY infinite, and each
    hidden unit's gradient infinite with the sign of the weight, not NaN."""
    params, X, U = problem(widths, B, seed=9)
    params[-1][1][i] = np.inf
    s = make_gpu(widths, params, B)
    s.train_step(padded_from(X), padded_from(U))
    torch.cuda.synchronize()
    _, gb = s.get_grads(len(widths) - 3)
    A = X.astype(np.float64)
    for W, b in params[:-1]:
        A = np.maximum(A @ W.T + b, 0.0)
    Wi = params[-1][0][i]
    active = A.max(axis=0) > 1e-2 * A.max()          # units that bf16 rounding leaves active in some row
    assert active.sum() >= 4 and active[i % widths[-2]]       # the unit whose weight column holds the bias copy
    assert np.array_equal(gb[active], np.sign(Wi[active]) * np.inf), gb
    s.close()
