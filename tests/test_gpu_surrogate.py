"""GPU surrogate against the fp64 oracle: initialisation (bit-exact), one train
step (loss, every gradient, parameters after Adam) over shapes that span
several tiles, ragged edges, split-K and the small-K first layer; prediction;
100 online steps on the 16x16 workload and on the 100x100 workload at its
full shape (slots bit-exact, loss, gradients and parameters within 1e-3
relative L2).  Gradients are also held element by element: every entry
within the tolerance times the largest reference entry."""
import numpy as np
import pytest
import torch

from fixtures import configs, heat
from oracle import mlp, runner

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def rel(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def elementwise(a, b):
    """Largest entry difference relative to the largest reference entry."""
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.max(np.abs(a - b))) / max(float(np.max(np.abs(b))), 1e-30)


def close(a, b, tol):
    """Relative L2 within tol and every element within tol of the largest
    reference entry (so that one wrong output unit among thousands fails)."""
    return rel(a, b) < tol and elementwise(a, b) < tol


def padded_from(arr):
    rows, d = arr.shape
    ld = (d + 3) // 4 * 4
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
    if widths[0] == 6:
        X = np.concatenate([rng.uniform(100, 500, (B, 5)), rng.uniform(0.01, 1.0, (B, 1))], axis=1)
        U = rng.uniform(100, 500, (B, widths[-1]))
    else:
        X = rng.normal(size=(B, widths[0]))
        U = rng.normal(size=(B, widths[-1]))
    return params, X.astype(np.float32), U.astype(np.float32)


def make_gpu(widths, params, B, flags=0):
    from paper_2309_16743_amd import Surrogate
    s = Surrogate(widths, max_batch=B, seed=0, flags=flags)
    for l, (W, b) in enumerate(params):
        s.set_params(l, W.astype(np.float32), b.astype(np.float32))
    return s


SHAPES = [
    ((6, 64, 64, 256), 32),          # the 16x16 workload's net
    ((6, 37, 50, 123), 45),          # ragged widths and batch
    ((6, 256, 256, 1000), 300),      # several tiles, split-K output input-gradient
    ((6, 128, 4000), 64),            # two layers, wide output
    ((20, 48, 30), 17),              # first layer through the GEMM path
    ((6, 10), 9),                    # single layer
    ((6, 256, 256, 10000), 1024),    # the 100x100 workload's net at its batch
    ((6, 8, 1), 1),                  # one sample, one output
    ((6, 300, 300, 7), 2),           # two samples, hidden widths past one tile
    # output products on three bf16 terms: every tile shape, ragged edges
    ((6, 200, 150, 70001), 20),      # 32 x 256 forward and input gradient, 512 splits
    ((6, 70, 131, 66000), 50),       # 64 x 256 forward and input gradient
    ((6, 90, 150, 13501), 300),      # 64 x 128 forward, 128 x 128 gradients, both split
    ((6, 200, 150, 40003), 200),     # unsplit weight gradient with Adam in its epilogue
    ((6, 60, 50, 20005), 250),       # gradients 50 units wide: 64 x 64 tiles
    ((6, 300, 437, 6561), 331),      # 64 x 64 forward, no dimension a multiple of 16
    ((24, 9001), 1000),              # single layer: the caller's unpadded x as an operand
]


@pytest.mark.parametrize("widths,B", SHAPES)
def test_one_train_step(widths, B):
    """Kept gradients: loss, every gradient and every parameter after Adam
    against the oracle.  Fused output-layer Adam (the default): the same
    parameters and Adam moments bit for bit (same gradient sums, same Adam
    arithmetic), the output bias gradient still readable, its weight gradient
    refused."""
    from paper_2309_16743_amd import OT_SURROGATE_KEEP_GRADS, OTError
    print(f"one train step widths={widths} B={B}", flush=True)
    params, X, U = problem(widths, B, seed=sum(widths) + B)
    s = make_gpu(widths, params, B, flags=OT_SURROGATE_KEEP_GRADS)
    f = make_gpu(widths, params, B)
    Xd, Ud = padded_from(X), padded_from(U)
    loss, loss_f = torch.zeros(1, device=DEV), torch.zeros(1, device=DEV)
    s.train_step(Xd, Ud, loss=loss)
    f.train_step(Xd, Ud, loss=loss_f)
    torch.cuda.synchronize()
    o_loss, o_grads = mlp.loss_and_grads(params, X.astype(np.float64), U.astype(np.float64))
    o_new = mlp.Adam(lr=1e-3).step(params, o_grads)
    assert abs(loss.item() - o_loss) / o_loss < 1e-5
    assert loss_f.item() == loss.item()
    L = len(widths) - 1
    for l in range(L):
        gW, gb = s.get_grads(l)
        assert close(gW, o_grads[l][0], 1e-4), (l, rel(gW, o_grads[l][0]))
        assert close(gb, o_grads[l][1], 1e-4), (l, rel(gb, o_grads[l][1]))
        W, b = s.get_params(l)
        assert rel(W, o_new[l][0]) < 1e-4 and rel(b, o_new[l][1]) < 1e-4
        Wf, bf = f.get_params(l)
        assert np.array_equal(Wf, W) and np.array_equal(bf, b), l
        (mW, mb), (vW, vb), t = s.get_adam_state(l)
        (mWf, mbf), (vWf, vbf), tf = f.get_adam_state(l)
        assert t == tf == 1
        for a, c in ((mWf, mW), (mbf, mb), (vWf, vW), (vbf, vb)):
            assert np.array_equal(a, c), l
    fused_out = not (L == 1 and widths[0] <= 16)   # a small-K single layer stores its gradient
    if fused_out:
        with pytest.raises(OTError):
            f.get_grads(L - 1)
    _, gb = s.get_grads(L - 1)
    assert np.array_equal(f.get_grads(L - 1, weights=False)[1], gb)
    s.close()
    f.close()


@pytest.mark.parametrize("widths,n", [((6, 64, 64, 256), 50), ((6, 37, 50, 123), 77), ((20, 48, 30), 5)])
def test_predict(widths, n):
    params, X, _ = problem(widths, n, seed=3)
    s = make_gpu(widths, params, 32)          # n above max_batch exercises the row chunking
    Y = padded_from(np.zeros((n, widths[-1]), np.float32))
    s.predict(padded_from(X), Y)
    torch.cuda.synchronize()
    ref = mlp.predict(params, X.astype(np.float64))
    assert rel(Y.cpu().numpy(), ref) < 1e-5
    s.close()


@pytest.mark.parametrize("widths,seed", [((6, 64, 64, 256), 1), ((6, 37, 50, 123), 7)])
def test_init_matches_oracle_bit_exact(widths, seed):
    from paper_2309_16743_amd import Surrogate
    s = Surrogate(widths, seed=seed, max_batch=8)
    ref = mlp.init_params(widths, seed)
    for l in range(len(widths) - 1):
        W, b = s.get_params(l)
        assert np.array_equal(W.astype(np.float64), ref[l][0])
        assert np.array_equal(b.astype(np.float64), ref[l][1])
    s.close()


def test_tiny_workload_100_steps():
    """16x16 heat fields, 6-64-64-256, batch 32, C 64, T 32: the schedule of the
    first workload; gradients compared at steps 1 and 100."""
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    from paper_2309_16743_amd import OT_SURROGATE_KEEP_GRADS
    ref = runner.run(w, inputs, fields, n_steps=100, keep_grads=(1, 100))
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100, flags=OT_SURROGATE_KEEP_GRADS)
    grads1 = None
    while tr.steps_done < 100:
        tr.iterate()
        if tr.steps_done == 1 and grads1 is None:
            grads1 = [tr.sur.get_grads(l) for l in range(3)]
    torch.cuda.synchronize()
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    losses = tr.loss_log.cpu().numpy()
    assert rel(losses, ref["losses"]) < 1e-3
    grads100 = [tr.sur.get_grads(l) for l in range(3)]
    for l in range(3):
        for i in range(2):
            assert close(grads1[l][i], ref["grads"][1][l][i], 1e-3)
            assert rel(grads100[l][i], ref["grads"][100][l][i]) < 1e-3    # L2 after 99 Adam steps
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    st = tr.res.stats()
    assert st["total_evicted"] == ref["reservoir"].total_evicted == 16
    tr.close()


def test_tiny_workload_100_steps_fused():
    """The same schedule with the output layer's Adam fused into its gradient
    GEMM (the default): slots bit-exact, loss series and final parameters
    within 1e-3 relative L2 of the oracle."""
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    ref = runner.run(w, inputs, fields, n_steps=100)
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100)
    tr.run(100)
    torch.cuda.synchronize()
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < 1e-3
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    tr.close()


def test_tiny_workload_graph_replayed_train_step():
    """The 16x16 schedule with the train step captured once as a HIP graph
    (Adam's step counter in device memory) and replayed for every step, the
    reservoir's calls and the log copies eager between the replays: slots,
    every step's loss and the final parameters and Adam state equal those of
    the eager run bit for bit (the step's arguments do not change between
    replays, and both modes form Adam's bias corrections the same way), and
    the oracle's within 1e-3."""
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    ref = runner.run(w, inputs, fields, n_steps=60)
    runs = {}
    for graph in (False, True):
        tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                           torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                           w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=60, graph=graph)
        while tr.steps_done < 60:
            tr.iterate()
            if tr.steps_done % 7 == 0:
                torch.cuda.synchronize()          # host synchronisations between replays
        torch.cuda.synchronize()
        if graph:
            assert tr._graph is not None
        runs[graph] = (tr.slot_log.cpu().numpy(), tr.loss_log.cpu().numpy(),
                       [tr.sur.get_params(l) for l in range(3)], [tr.sur.get_adam_state(l) for l in range(3)])
        if graph:
            tr.sur.set_device_step(False)
            assert tr.sur.get_adam_state(0)[2] == 60
        tr.close()
    (s0, l0, p0, a0), (s1, l1, p1, a1) = runs[False], runs[True]
    assert np.array_equal(s0, s1)
    assert np.array_equal(l0, l1)
    for l in range(3):
        assert np.array_equal(p0[l][0], p1[l][0]) and np.array_equal(p0[l][1], p1[l][1])
        (m0, v0, t0), (m1, v1, t1) = a0[l], a1[l]
        assert t0 == t1 == 60
        assert all(np.array_equal(x, y) for x, y in zip(m0 + v0, m1 + v1))
    for i in range(60):
        assert np.array_equal(s1[i], ref["slots"][i]), i
    assert rel(l1, ref["losses"]) < 1e-3
    for l in range(3):
        assert rel(p1[l][0], ref["params"][l][0]) < 1e-3


def test_tiny_workload_overlapped_streams():
    """The 16x16 schedule with the reservoir on its own stream and two batch
    buffers (the draw of batch i + 1 overlaps train step i): the same slots
    bit for bit and the same losses as the oracle."""
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    ref = runner.run(w, inputs, fields, n_steps=100)
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100, overlap=True)
    tr.run(100)
    torch.cuda.synchronize()
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < 1e-3
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    tr.close()


def test_tiny_workload_schedule_validation_histogram():
    """The 16x16 schedule with the learning rate halved every 640 trained
    samples down to 2.5e-4 and validation every 25 steps on two held-out
    simulations (surrogate_eval_loss): slots bit-exact, loss series, final
    parameters and validation losses within 1e-3 relative of the oracle; the
    repetition histogram bit-exact."""
    from paper_2309_16743_amd.online import HalvingLR, OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    Xv = heat.sample_parameters(2, 99)
    iv, fv = heat.inputs_for(Xv, w.tau).reshape(-1, 6), heat.heat_fields(Xv, w.grid, w.tau).reshape(-1, 256)
    ref = runner.run(w, inputs, fields, n_steps=100, lr_halving=(640, 2.5e-4), validation=(iv, fv, 25))
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100,
                       lr_schedule=HalvingLR(1e-3, 640, 2.5e-4))
    ivd, fvd = padded_from(iv), padded_from(fv)
    val = {}
    while tr.steps_done < 100:
        if tr.iterate() and tr.steps_done % 25 == 0:
            val[tr.steps_done] = tr.validate(ivd, fvd, torch.zeros(1, device=DEV))
    torch.cuda.synchronize()
    assert tr.lr == 2.5e-4
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < 1e-3
    for k, v in ref["val_losses"].items():
        assert abs(val[k].item() - v) / v < 1e-3, (k, val[k].item(), v)
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    h = tr.repetition_histogram()
    assert np.array_equal(h, runner.repetition_histogram(ref["reservoir"], len(h)))
    tr.close()


@pytest.mark.parametrize("widths,n,bf16", [((6, 64, 64, 256), 200, False), ((6, 37, 50, 123), 77, False),
                                           ((6, 100, 77, 1001), 150, True)])
def test_eval_loss(widths, n, bf16):
    """surrogate_eval_loss over more rows than the workspace (chunked) against
    the oracle's MSE of its prediction; parameters untouched."""
    from paper_2309_16743_amd import OT_BF16, OT_FP32, Surrogate
    params, X, U = problem(widths, n, seed=21)
    s = Surrogate(widths, precision=OT_BF16 if bf16 else OT_FP32, max_batch=64, seed=0)
    for l, (W, b) in enumerate(params):
        s.set_params(l, W.astype(np.float32), b.astype(np.float32))
    loss = torch.zeros(1, device=DEV)
    s.eval_loss(padded_from(X), padded_from(U), loss)
    torch.cuda.synchronize()
    ref = mlp.mse(mlp.predict(params, X.astype(np.float64), bf16=bf16), U.astype(np.float64))
    assert abs(loss.item() - ref) / ref < (1e-3 if bf16 else 1e-5), (loss.item(), ref)
    for l in range(len(widths) - 1):
        W, b = s.get_params(l)
        assert np.array_equal(W, params[l][0].astype(np.float32))
    s.close()


@pytest.mark.parametrize("widths,B,bf16", [((6, 256, 256, 10000), 1024, False), ((6, 100, 77, 1001), 50, False),
                                           ((6, 512, 512, 20000), 512, True), ((6, 64, 64, 256), 32, True)])
def test_train_step_rows_equals_gathered_rows(widths, B, bf16):
    """surrogate_train_step_rows (targets read in place from a larger array
    through row indices) against surrogate_train_step on the same rows
    gathered: loss and every parameter bit for bit, two steps in a row; an
    index past the array is clamped to its last row."""
    from paper_2309_16743_amd import OT_BF16, OT_FP32, Surrogate
    print(f"train_step_rows widths={widths} B={B} bf16={bf16}", flush=True)
    rng = np.random.default_rng(B)
    params, X, _ = problem(widths, B, seed=B + 1)
    n_rows = 3 * B + 7
    D = widths[-1]
    ldu = (D + 63) // 64 * 64
    slab = torch.from_numpy(rng.uniform(100, 500, (n_rows, ldu)).astype(np.float32)).to(DEV)
    rows = rng.integers(0, n_rows, B).astype(np.int32)
    rows[0] = n_rows - 1
    prec = OT_BF16 if bf16 else OT_FP32
    a = Surrogate(widths, precision=prec, max_batch=B, seed=0)
    g = Surrogate(widths, precision=prec, max_batch=B, seed=0)
    for l, (W, b) in enumerate(params):
        a.set_params(l, W.astype(np.float32), b.astype(np.float32))
        g.set_params(l, W.astype(np.float32), b.astype(np.float32))
    Xd = padded_from(X)
    rows_d = torch.from_numpy(rows).to(DEV)
    gathered = torch.zeros(B, ldu, device=DEV)[:, :D]
    gathered.copy_(slab[rows_d.long(), :D])
    ev = torch.cuda.Event()
    la, lg = torch.zeros(1, device=DEV), torch.zeros(1, device=DEV)
    for _ in range(2):
        a.train_step_rows(Xd, slab.data_ptr(), ldu, rows_d, n_rows, loss=la, targets_read=ev)
        g.train_step(Xd, gathered, loss=lg)
    torch.cuda.synchronize()
    assert la.item() == lg.item()
    for l in range(len(widths) - 1):
        Wa, ba = a.get_params(l)
        Wg, bg = g.get_params(l)
        assert np.array_equal(Wa, Wg) and np.array_equal(ba, bg), l
    # clamping: an index past the array reads its last row
    bad = rows_d.clone()
    bad[0] = n_rows + 1000
    lc = torch.zeros(1, device=DEV)
    c = Surrogate(widths, precision=prec, max_batch=B, seed=0)
    for l, (W, b) in enumerate(params):
        c.set_params(l, W.astype(np.float32), b.astype(np.float32))
    c.train_step_rows(Xd, slab.data_ptr(), ldu, bad, n_rows, loss=lc)
    d = Surrogate(widths, precision=prec, max_batch=B, seed=0)
    for l, (W, b) in enumerate(params):
        d.set_params(l, W.astype(np.float32), b.astype(np.float32))
    ld = torch.zeros(1, device=DEV)
    d.train_step_rows(Xd, slab.data_ptr(), ldu, rows_d, n_rows, loss=ld)
    torch.cuda.synchronize()
    assert lc.item() == ld.item()
    for s in (a, g, c, d):
        s.close()


@pytest.mark.parametrize("overlap", [False, True])
def test_tiny_workload_fused_and_gathered_targets_agree(overlap):
    """The 16x16 schedule with the targets read in place from the reservoir
    (the default) and with the batch's rows gathered first: the same slots,
    losses and parameters bit for bit."""
    from paper_2309_16743_amd.online import OnlineTrainer
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = torch.from_numpy(heat.inputs_for(X, w.tau)).to(DEV)
    fields = torch.from_numpy(heat.heat_fields(X, w.grid, w.tau)).to(DEV)
    out = []
    for fused in (True, False):
        tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau, inputs, fields,
                           w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100, overlap=overlap,
                           fused_targets=fused)
        tr.run(100)
        torch.cuda.synchronize()
        out.append((tr.slot_log.cpu().numpy(), tr.loss_log.cpu().numpy(),
                    [tr.sur.get_params(l) for l in range(3)]))
        tr.close()
    (sa, la, pa), (sg, lg, pg) = out
    assert np.array_equal(sa, sg) and np.array_equal(la, lg)
    for (Wa, ba), (Wg, bg) in zip(pa, pg):
        assert np.array_equal(Wa, Wg) and np.array_equal(ba, bg)


@pytest.mark.parametrize("policy_name", ["reservoir", "fifo", "firo"])
@pytest.mark.parametrize("overlap", [False, True])
def test_tiny_schedule_to_drain_per_policy(policy_name, overlap):
    """The whole 16x16 schedule through each buffer policy, then the end of
    reception and the drain with training on every batch (the last one may be
    short): slots of every batch bit-exact, batch sizes equal, loss series and
    final parameters within 1e-3 relative of the oracle's run_to_drain."""
    from oracle.buffers import FIFOBuffer, FIROBuffer
    from oracle.reservoir import Reservoir
    from paper_2309_16743_amd import OT_POLICY_FIFO, OT_POLICY_FIRO, OT_POLICY_RESERVOIR
    from paper_2309_16743_amd.online import OnlineTrainer
    cls, policy = {"reservoir": (Reservoir, OT_POLICY_RESERVOIR), "fifo": (FIFOBuffer, OT_POLICY_FIFO),
                   "firo": (FIROBuffer, OT_POLICY_FIRO)}[policy_name]
    print(f"schedule to drain policy={policy_name} overlap={overlap}", flush=True)
    w = configs.TINY
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    ref = runner.run_to_drain(w, inputs, fields,
                              cls(w.capacity, w.threshold, inputs.shape[-1], fields.shape[-1], w.reservoir_seed))
    n = len(ref["losses"])
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=n, overlap=overlap, policy=policy)
    for _ in range(w.n_chunks):
        tr.iterate()
    torch.cuda.synchronize()
    tr.res.end_reception()
    while tr.sample_and_train():
        pass
    torch.cuda.synchronize()
    assert tr.steps_done == n
    slots = tr.slot_log.cpu().numpy()
    for i in range(n):
        k = ref["sizes"][i]
        assert np.array_equal(slots[i][:k], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < 1e-3
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    tr.close()


def test_timing_hooks_cover_the_timed_calls():
    """The profiling hooks behind the benchmark's per-kernel table: every
    output-layer GEMM phase is timed once per step and the reservoir's phases
    once per call, with positive durations; calls past max_steps are not
    counted and results are unchanged by timing."""
    from paper_2309_16743_amd import Reservoir, Surrogate, _abi
    widths, B = (6, 64, 64, 256), 32
    params, X, U = problem(widths, B, seed=3)
    s, ref = make_gpu(widths, params, B), make_gpu(widths, params, B)
    Xd, Ud = padded_from(X), padded_from(U)
    s.timing_begin(list(_abi.SURROGATE_PHASES), 3)
    for _ in range(5):
        s.train_step(Xd, Ud)
        ref.train_step(Xd, Ud)
    r = s.timing_end()
    for p in ("fwd_output", "wgrad_output", "igrad_output"):
        assert r[p][1] == 3 and r[p][0] > 0, (p, r.get(p))
    for l in range(3):
        W, b = s.get_params(l)
        Wr, br = ref.get_params(l)
        assert np.array_equal(W, Wr) and np.array_equal(b, br)
    s.close()
    ref.close()
    res = Reservoir(64, 8, 6, 256, 1)
    res.timing_begin(list(_abi.RESERVOIR_PHASES), 10)
    res.put(padded_from(X), padded_from(U))
    slots = torch.empty(16, dtype=torch.int32, device=DEV)
    xb, ub = padded_from(np.zeros((16, 6), np.float32)), padded_from(np.zeros((16, 256), np.float32))
    res.sample_batch(16, slots, x_out=xb, u_out=ub)
    torch.cuda.synchronize()
    rr = res.timing_end()
    for p in _abi.RESERVOIR_PHASES:
        assert rr[p][1] == 1 and rr[p][0] > 0, (p, rr.get(p))
    res.close()


def test_full_net_online_schedule_with_evictions():
    """The 100x100 workload's net (6-256-256-10,000 fp32) and batch (1024)
    through the online loop as the benchmark runs it (two streams, targets
    read in place from the reservoir), with a reservoir reduced to 1200 slots
    so that evictions start within the run: 20 train steps, slots bit-exact,
    loss series and final parameters within 1e-3 relative L2 of the oracle."""
    import dataclasses
    from paper_2309_16743_amd.online import OnlineTrainer
    w = dataclasses.replace(configs.HEAT100, n_sims=40, wave=40, capacity=1200, threshold=1024)
    print(f"full-net online schedule C={w.capacity} T={w.threshold} B={w.batch}", flush=True)
    X = heat.sample_parameters(w.n_sims, w.data_seed)
    inputs = heat.inputs_for(X, w.tau)
    fields = heat.heat_fields(X, w.grid, w.tau)
    n = 20
    ref = runner.run(w, inputs, fields, n_steps=n)
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=n, overlap=True)
    tr.run(n)
    torch.cuda.synchronize()
    assert tr.res.stats()["total_evicted"] > 0
    slots = tr.slot_log.cpu().numpy()
    for i in range(n):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    assert rel(tr.loss_log.cpu().numpy(), ref["losses"]) < 1e-3
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3
    tr.close()


_HEAT_FULL = {}


def heat_full_shape_reference():
    """Inputs and the oracle's 100-step run of the full-shape 100x100 workload
    (computed once for both parametrisations of the test below)."""
    if not _HEAT_FULL:
        import dataclasses
        w = dataclasses.replace(configs.HEAT100, n_sims=300)
        X = heat.sample_parameters(w.n_sims, w.data_seed)
        assert np.array_equal(X, heat.sample_parameters(configs.HEAT100.n_sims, w.data_seed)[:w.n_sims])
        inputs = heat.inputs_for(X, w.tau)
        fields = heat.heat_fields(X, w.grid, w.tau)
        ref = runner.run(w, inputs, fields, n_steps=100, keep_grads=(1, 100))
        ref["N"] = ref.pop("reservoir").N
        _HEAT_FULL.update(w=w, inputs=inputs, fields=fields, ref=ref)
    return _HEAT_FULL["w"], _HEAT_FULL["inputs"], _HEAT_FULL["fields"], _HEAT_FULL["ref"]


@pytest.mark.parametrize("flags", ["keep_grads", "fused"])
def test_heat_workload_full_shape_100_steps(flags):
    """The 100x100 workload at its full shape: 6-256-256-10,000 fp32, batch
    1024, a reservoir of 100,000 samples with threshold 16,667, chunks of the
    100 concurrent simulations' time step, through the two-stream loop with
    the targets read in place (as bench.py runs it), for 100 train steps (the
    266 iterations they take stream the first 300 simulations of the
    ensemble).  Slots bit-exact at every step; loss series and final
    parameters within 1e-3 relative L2 of the oracle, every loss within 1e-3
    of its own; with kept gradients, the gradients of step 1 and of step 100
    within 1e-3 in L2 and element-wise, those of step 100 against the
    oracle's gradients at the path's own parameters after step 99 on the
    step's batch; with the output layer's Adam fused (the benchmark's path)
    the same slots, losses and parameters."""
    from paper_2309_16743_amd import OT_SURROGATE_KEEP_GRADS
    from paper_2309_16743_amd.online import OnlineTrainer
    print(f"100x100 workload at full shape, 100 steps ({flags})", flush=True)
    w, inputs, fields, ref = heat_full_shape_reference()
    assert (w.capacity, w.threshold, w.batch, w.wave) == (100_000, 16_667, 1024, 100)
    assert ref["iterations"] == 266
    keep = flags == "keep_grads"
    tr = OnlineTrainer(w.widths, w.batch, w.capacity, w.threshold, w.wave, w.tau,
                       torch.from_numpy(inputs).to(DEV), torch.from_numpy(fields).to(DEV),
                       w.reservoir_seed, w.init_seed, lr=w.lr, record_steps=100, overlap=True,
                       flags=OT_SURROGATE_KEEP_GRADS if keep else 0)
    grads1 = params99 = None
    while tr.steps_done < 100:
        tr.iterate()
        if keep and tr.steps_done == 1 and grads1 is None:
            grads1 = [tr.sur.get_grads(l) for l in range(3)]
        if keep and tr.steps_done == 99 and params99 is None:
            params99 = [tuple(a.astype(np.float64) for a in tr.sur.get_params(l)) for l in range(3)]
    torch.cuda.synchronize()
    assert tr.iteration == 266
    slots = tr.slot_log.cpu().numpy()
    for i in range(100):
        assert np.array_equal(slots[i], ref["slots"][i]), i
    losses = tr.loss_log.cpu().numpy()
    assert rel(losses, ref["losses"]) < 1e-3
    assert np.max(np.abs(losses - ref["losses"]) / np.array(ref["losses"])) < 1e-3
    if keep:
        # Step 100's gradients are held against the oracle's gradients of the
        # same batch at the path's own parameters after step 99: the 99 Adam
        # steps before it leave the two trajectories apart in the last bits,
        # and near-zero pre-activations then fall on different sides of the
        # ReLU, which moves the layer-1 gradient (its inputs are raw
        # temperatures of 100-500) by about 1.6e-3 in L2 even between the
        # oracle and the oracle with its stored state rounded to fp32.  The
        # distance to the oracle's own step 100 is printed, and bounded by
        # four times that sensitivity.
        grads100 = [tr.sur.get_grads(l) for l in range(3)]
        xb, ub = ref["batches"][100]
        assert xb.shape == (1024, 6) and ub.shape == (1024, 10_000)
        _, o100 = mlp.loss_and_grads(params99, xb, ub)
        for l in range(3):
            for i in range(2):
                g1, o1 = grads1[l][i], ref["grads"][1][l][i]
                assert close(g1, o1, 1e-3), (1, l, i, rel(g1, o1), elementwise(g1, o1))
                g, o = grads100[l][i], o100[l][i]
                assert close(g, o, 1e-3), (100, l, i, rel(g, o), elementwise(g, o))
                t = ref["grads"][100][l][i]
                print(f"  step 100 layer {l} {'dW' if i == 0 else 'db'}: at the path's parameters rel L2 "
                      f"{rel(g, o):.2e} element-wise {elementwise(g, o):.2e}; against the oracle's trajectory "
                      f"rel L2 {rel(g, t):.2e}", flush=True)
                assert rel(g, t) < 6.4e-3, (100, l, i, rel(g, t))
    for l in range(3):
        W, b = tr.sur.get_params(l)
        assert rel(W, ref["params"][l][0]) < 1e-3 and rel(b, ref["params"][l][1]) < 1e-3, l
    st = tr.res.stats()
    assert st["n"] == ref["N"] == 26_600 and st["total_draws"] == 100 * 1024
    tr.close()


@pytest.mark.parametrize("value", [2.0 ** 70, 3.3e38, np.inf, np.nan])
def test_predict_beyond_split_range(value):
    """A product on three bf16 terms whose operands hold a value beyond the
    range of the split (or infinity, NaN): the same finite and non-finite
    outputs as fp32 arithmetic, the other outputs unchanged."""
    widths, B = (6, 64, 64, 20000), 200
    params, X, _ = problem(widths, B, seed=11)
    W, b = params[-1]
    W[:, 5] = np.where(np.arange(len(W)) % 2 == 0, W[:, 5], 1.0)      # exact in bf16: further terms are zero
    W[777, 5] = value
    W[778, 5] = -value
    s = make_gpu(widths, params, B)
    Y = padded_from(np.zeros((B, widths[-1]), np.float32))
    s.predict(padded_from(X), Y)
    torch.cuda.synchronize()
    got = Y.cpu().numpy()
    A = X.astype(np.float64)
    for Wl, bl in params[:-1]:
        A = np.maximum(A @ Wl.T + bl, 0.0)
    A = A.astype(np.float32).astype(np.float64)
    with np.errstate(all="ignore"):
        ref = (A @ W.astype(np.float32).astype(np.float64).T + b).astype(np.float32)
        # a term that overflows fp32 makes the sum infinite whatever follows
        over = np.abs(A[:, 5] * np.float64(np.float32(value))) > np.finfo(np.float32).max
    if np.isfinite(value):
        ref[over, 777], ref[over, 778] = np.inf, -np.inf
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.array_equal(np.sign(got[~fin & ~np.isnan(ref)]), np.sign(ref[~fin & ~np.isnan(ref)]))
    # fp32 sums of 64 terms, relative to the largest one of the row
    scale = np.maximum(np.abs(ref), np.abs(A).max() * np.minimum(np.abs(np.nan_to_num(W, posinf=0.0)).max(axis=1), 1e38))
    assert np.all(np.abs(got - ref)[fin] <= 64 * 2.0 ** -24 * scale[fin])
    s.close()


@pytest.mark.parametrize("value", [2.0 ** 90, 3.3e38, np.inf, np.nan])
@pytest.mark.parametrize("flags", ["keep_grads", "fused"])
@pytest.mark.parametrize("widths,B", [((24, 9001), 1000),            # weight gradient in splits
                                      ((6, 64, 160, 40000), 200)])   # unsplit; input gradient in splits
def test_gradients_beyond_split_range(widths, B, flags, value):
    """A target column far out of range makes one column of dY reach beyond the
    range of the bf16 split (or infinity, NaN) in the gradient products: the
    weight rows, moments and bias entries of every other output are those of
    fp32 arithmetic, and so, while they are finite, are the output's own row and the
    hidden layers' gradients."""
    from paper_2309_16743_amd import OT_SURROGATE_KEEP_GRADS
    L, n = len(widths) - 1, 1234
    params, X, U = problem(widths, B, seed=12)
    U[:, n] = value
    keep = flags == "keep_grads"
    s = make_gpu(widths, params, B, flags=OT_SURROGATE_KEEP_GRADS if keep else 0)
    s.train_step(padded_from(X), padded_from(U), loss=torch.zeros(1, device=DEV))
    torch.cuda.synchronize()
    clean = U.copy()
    clean[:, n] = 1.0
    _, grads = mlp.loss_and_grads(params, X.astype(np.float64), clean.astype(np.float64))
    new = mlp.Adam(lr=1e-3).step(params, grads)
    others = np.arange(widths[-1]) != n
    W, b = s.get_params(L - 1)
    (mW, mb), _, _ = s.get_adam_state(L - 1)
    assert close(mW[others], 0.1 * grads[-1][0][others], 1e-4) and close(mb[others], 0.1 * grads[-1][1][others], 1e-4)
    assert rel(W[others], new[-1][0][others]) < 1e-4 and rel(b[others], new[-1][1][others]) < 1e-4
    if keep:
        gW, gb = s.get_grads(L - 1)
        assert close(gW[others], grads[-1][0][others], 1e-4) and close(gb[others], grads[-1][1][others], 1e-4)
    if np.isfinite(value):
        # fp32 sums of the B rows: products of dY (about value / (B D)) stay finite
        _, full = mlp.loss_and_grads(params, X.astype(np.float64), U.astype(np.float64))
        assert close(mW[n], 0.1 * full[-1][0][n], 1e-4)
        for l in range(L - 1):
            gW, gb = s.get_grads(l)
            assert close(gW, full[l][0], 1e-4) and close(gb, full[l][1], 1e-4), l
    else:
        assert not np.isfinite(mW[n]).any() and not np.isfinite(mb[n])
    s.close()


def test_calls_after_a_step_too_large_for_memory():
    """A train step whose workspaces do not fit the device is refused before
    anything is enqueued; predictions, evaluations and smaller steps after it get
    workspaces of their own again."""
    from paper_2309_16743_amd import load
    from paper_2309_16743_amd._abi import OT_E_NOMEM
    widths, B = (6, 64, 64, 1_000_000), 8
    params, X, U = problem(widths, B, seed=13)
    s = make_gpu(widths, params, B)
    x, u = padded_from(X), padded_from(U)
    y = [padded_from(np.zeros((B, widths[-1]), np.float32)) for _ in range(2)]
    losses = torch.zeros(2, device=DEV)
    for i in range(2):
        s.predict(x, y[i])
        s.eval_loss(x, u, losses[i:i + 1])
        torch.cuda.synchronize()
        if i == 0:              # 2^20 rows of dY alone would be 4 TB; x and u are not read
            assert load().surrogate_train_step(s.handle, x.data_ptr(), 8, u.data_ptr(), widths[-1], 1 << 20, None,
                                               None) == OT_E_NOMEM
    assert torch.equal(y[0], y[1]) and losses[0].item() == losses[1].item()
    s.train_step(x, u)
    torch.cuda.synchronize()
    assert s.get_adam_state(0)[2] == 1
    s.close()
