"""GPU BF16-MFMA MLP kernels against the FP64 oracle MLP (which emulates
the same bfloat16 rounding points)."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_05386_amd import rt
    return rt, torch, rt.Tracer(0)


def _params(torch, n, scale=1.0):
    p = np.stack([mlp.init_params(10 + i) for i in range(n)]) * scale
    rng = np.random.default_rng(1)
    for i in range(n):   # non-zero biases
        for k, (o, _) in zip(range(4), mlp.SIZES):
            mlp.split(p[i])[2 * k + 1][:] = rng.normal(0, 0.1, size=o)
    pt = torch.tensor(p, dtype=torch.float32, device="cuda")
    return p, pt, pt.to(torch.bfloat16)


# batches that are multiples of 8 take the vector-staged backward products,
# multiples of 128 the split-K weight gradient and the LDS-staged epilogue
# (264: a ragged last tile of 8 rows), the others the element-wise ones
@pytest.mark.parametrize("n,batch", [(3, 37), (2, 300), (1, 1), (2, 264), (1, 1024), (3, 512)])
def test_mlp_forward_backward_match_oracle(env, n, batch):
    rt, torch, tr = env
    say("mlp fwd/bwd n_nets=%d batch=%d" % (n, batch))
    p, pt, pb = _params(torch, n)
    rng = np.random.default_rng(2)
    x = rng.normal(size=(n, batch, 6)).astype(np.float32)
    dy = rng.normal(size=(n, batch, 6)).astype(np.float32)
    work = tr.mlp_work(n, batch)
    y = tr.mlp_fwd(pb, pt, torch.tensor(x, device="cuda"), work).cpu().numpy()
    g = tr.mlp_bwd(pb, pt, torch.tensor(dy, device="cuda"), work).cpu().numpy()
    p32 = p.astype(np.float32).astype(np.float64)
    worst_f = worst_b = 0.0
    for i in range(n):
        yr, _ = mlp.forward(p32[i], x[i].astype(np.float64), bf16=True)
        ef = np.abs(y[i] - yr).max() / max(1.0, np.abs(yr).max())
        worst_f = max(worst_f, ef)
        # the oracle rounds at the same bf16 points; what remains is FP32
        # accumulation order (measured worst 4.1e-6)
        assert ef <= 2e-5, (i, ef)
        gr = mlp.backward(p32[i], x[i].astype(np.float64), dy[i].astype(np.float64), bf16=True)
        for blk, (a, b) in enumerate(zip(mlp.split(g[i].astype(np.float64)), mlp.split(gr))):
            err = np.abs(a - b).max() / max(1e-3, np.abs(b).max())
            worst_b = max(worst_b, err)
            # backward operands are rounded to bf16 from FP32 values that
            # differ from the oracle's FP64 ones by accumulation order; an
            # element that lies that close to a rounding boundary goes to
            # the neighbouring bf16 value (2^-8 relative), so a sum of 256
            # terms can move by about one bf16 ulp of one term (measured
            # worst 9.8e-4 of the largest component)
            assert err <= 3e-3, (i, blk, err, np.abs(b).max())
    say("worst relative error: forward %.2e, backward %.2e" % (worst_f, worst_b))


@pytest.mark.parametrize("n,batch", [(2, 1024), (3, 264)])
def test_mlp_backward_is_deterministic(env, n, batch):
    """The weight gradients split K over the waves of a block and sum the
    partial tiles in a fixed order, the FP32 layers sum fixed row chunks in
    order: two backward passes give the same bits."""
    rt, torch, tr = env
    say("mlp backward determinism n_nets=%d batch=%d" % (n, batch))
    p, pt, pb = _params(torch, n)
    rng = np.random.default_rng(5)
    x = torch.tensor(rng.normal(size=(n, batch, 6)).astype(np.float32), device="cuda")
    dy = torch.tensor(rng.normal(size=(n, batch, 6)).astype(np.float32), device="cuda")
    out = []
    for _ in range(2):
        work = tr.mlp_work(n, batch)
        tr.mlp_fwd(pb, pt, x, work)
        out.append(tr.mlp_bwd(pb, pt, dy, work).cpu().numpy())
    assert np.array_equal(out[0], out[1])


def test_adamw_step(env):
    rt, torch, tr = env
    say("adamw")
    rng = np.random.default_rng(3)
    n = 1000
    p = rng.normal(size=n).astype(np.float32)
    m = rng.normal(size=n).astype(np.float32) * 0.1
    v = np.abs(rng.normal(size=n)).astype(np.float32) * 0.01
    g = rng.normal(size=n).astype(np.float32)
    P, M, V, G = (torch.tensor(a, device="cuda") for a in (p, m, v, g))
    PB = P.to(torch.bfloat16)
    lr, b1, b2, eps, wd, step = 1e-3, 0.9, 0.999, 1e-8, 0.01, 7
    tr.adamw(P, PB, M, V, G, lr, step, b1, b2, eps, wd)
    m2 = b1 * m + (1 - b1) * g
    v2 = b2 * v + (1 - b2) * g * g
    p2 = p - lr * ((m2 / (1 - b1 ** step)) / (np.sqrt(v2 / (1 - b2 ** step)) + eps) + wd * p)
    assert np.allclose(P.cpu().numpy(), p2, rtol=1e-5, atol=1e-6)
    assert np.allclose(PB.float().cpu().numpy(), p2, rtol=1e-2, atol=1e-3)


def test_training_reduces_loss(env):
    rt, torch, tr = env
    say("mlp training on a smooth 6->6 map")
    n, batch = 2, 512
    p, pt, pb = _params(torch, n, scale=0.5)
    rng = np.random.default_rng(4)
    x = torch.tensor(rng.uniform(-1, 1, size=(n, batch, 6)), dtype=torch.float32, device="cuda")
    t = torch.sin(2.0 * x) * 0.5 + x.roll(1, dims=2) * 0.3
    m = torch.zeros_like(pt)
    v = torch.zeros_like(pt)
    work = tr.mlp_work(n, batch)
    losses = []
    for step in range(1, 301):
        y = tr.mlp_fwd(pb, pt, x, work)
        diff = y - t
        losses.append(float((diff * diff).sum() / (n * batch)))
        g = tr.mlp_bwd(pb, pt, 2.0 * diff / batch, work)
        tr.adamw(pt, pb, m, v, g, 2e-3, step)
    say("loss", losses[0], "->", losses[-1])
    assert losses[-1] < 0.05 * losses[0]


@pytest.mark.parametrize("n,batch", [(2, 63), (2, 64), (2, 65), (1, 127), (1, 128), (1, 129), (5, 1000)])
def test_mlp_tile_edges(env, n, batch):
    """Batches about the 64-row tiles: forward and backward against the oracle
    within the bounds of test_mlp_forward_backward_match_oracle, and the work
    buffer of one batch used again with other rows (the padding rows of the
    last tile add nothing)."""
    rt, torch, tr = env
    say("mlp tile edges n_nets=%d batch=%d" % (n, batch))
    p, pt, pb = _params(torch, n)
    p32 = p.astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(batch)
    work = tr.mlp_work(n, batch)
    for scale in (3.0, 1.0):
        x = (scale * rng.normal(size=(n, batch, 6))).astype(np.float32)
        dy = rng.normal(size=(n, batch, 6)).astype(np.float32)
        y = tr.mlp_fwd(pb, pt, torch.tensor(x, device="cuda"), work).cpu().numpy()
        g = tr.mlp_bwd(pb, pt, torch.tensor(dy, device="cuda"), work).cpu().numpy()
    for i in range(n):
        yr, _ = mlp.forward(p32[i], x[i].astype(np.float64), bf16=True)
        assert np.abs(y[i] - yr).max() <= 2e-5 * max(1.0, np.abs(yr).max()), i
        gr = mlp.backward(p32[i], x[i].astype(np.float64), dy[i].astype(np.float64), bf16=True)
        for blk, (a, b) in enumerate(zip(mlp.split(g[i].astype(np.float64)), mlp.split(gr))):
            assert np.abs(a - b).max() <= 3e-3 * max(1e-3, np.abs(b).max()), (i, blk)


def test_grouped_forward_on_two_streams(env):
    """Grouped calls on two streams in turn, the group count growing between
    them: each result equals the same call made alone."""
    rt, torch, tr = env
    say("grouped forward on two streams")
    rng = np.random.default_rng(8)
    calls = []
    for n in (1, 3, 40, 2):
        _, pt, pb = _params(torch, n)
        rows = [int(r) for r in rng.integers(0, 150, n)]
        rows[0] = 65
        x = torch.tensor(rng.normal(size=(sum(rows), 6)).astype(np.float32), device="cuda")
        calls.append((pb, pt, x, rows))
    alone = [tr.mlp_fwd_grouped(*c).clone() for c in calls]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for k, c in enumerate(calls * 2):
        with torch.cuda.stream(streams[k % 2]):
            got.append(tr.mlp_fwd_grouped(*c))
    torch.cuda.synchronize()
    for k, y in enumerate(got):
        assert torch.equal(y, alone[k % len(calls)]), k


@pytest.mark.parametrize("n", [1, 255, 257, 6000, 16385, 65537])
def test_mse_partials(env, n):
    """The 64 partial sums of the loss: partial b holds the elements whose
    index / 256 is b modulo 64; a sum of k FP32 squares in any order is within
    (k + 2) 2^-24 of the exact one, relative."""
    rt, torch, tr = env
    say("mse partials n=%d" % n)
    rng = np.random.default_rng(n)
    y, t = (rng.normal(size=n).astype(np.float32) for _ in range(2))
    dy, part = tr.mse_grad(torch.tensor(y, device="cuda"), torch.tensor(t, device="cuda"), 7)
    d = (y - t).astype(np.float64)
    assert np.allclose(dy.cpu().numpy(), 2.0 * d / 7.0, rtol=4e-7, atol=0)
    b = np.arange(n) // 256 % 64
    ref = np.bincount(b, d * d, 64)
    k = np.bincount(b, minlength=64)
    assert (np.abs(part.cpu().numpy() - ref) <= (k + 2) * 2.0**-24 * ref).all()


def _plain_net(torch, **parts):
    """One network of zeros with the named parts (W1, b1, ..., b4) set."""
    p = np.zeros(mlp.N_PARAMS)
    names = ["%s%d" % (a, i) for i in (1, 2, 3, 4) for a in "Wb"]
    for k, v in parts.items():
        mlp.split(p)[names.index(k)][:] = v
    pt = torch.tensor(p[None], dtype=torch.float32, device="cuda")
    return pt, pt.to(torch.bfloat16)


@pytest.mark.parametrize("lo,hi", [(-80.0, 80.0), (-1e3, 1e3), (-1e37, -90.0)])
def test_activation_values(env, lo, hi):
    """SiLU and its derivative by themselves, on both sides of the range where
    the quotients are formed without a division: with W2 = W3 = 0 the last
    pre-activations are b3, and with one row and dy = e_0 the gradient of W4's
    first row is silu(b3), that of b3 is W4 silu'(b3).  The exponential's
    argument z log2(e) is rounded to FP32 and the hardware exponential adds an
    ulp: a relative error of at most (|z| + 2) 2^-23 in exp(-z), and a few
    ulp after that.  From -89 on exp(-z) overflows, and both are zero."""
    rt, torch, tr = env
    say("activations %g .. %g" % (lo, hi))
    z = np.linspace(lo, hi, 256).astype(np.float32)
    pt, pb = _plain_net(torch, b3=z, W4=np.eye(6, 1))
    x = torch.zeros((1, 1, 6), device="cuda")
    dy = torch.zeros((1, 1, 6), device="cuda")
    dy[..., 0] = 1.0
    work = tr.mlp_work(1, 1)
    y = tr.mlp_fwd(pb, pt, x, work).cpu().numpy()[0, 0]
    parts = mlp.split(tr.mlp_bwd(pb, pt, dy, work).cpu().numpy()[0].astype(np.float64))
    h, dz = parts[6][0], parts[5]
    z = z.astype(np.float64)
    with np.errstate(over="ignore"):
        e = np.exp(-z)
    far = z <= -89.0
    s = 1.0 / (1.0 + e)
    rel = (np.abs(z) + 6.0) * 2.0**-23
    assert (h[far] == 0.0).all() and (dz[far] == 0.0).all()
    ok = ~far
    assert (np.abs(h - z * s)[ok] <= (rel * np.abs(z) * s + 1e-38)[ok]).all()
    # s (1 + z (1 - s)): the terms by themselves, for they cancel
    assert (np.abs(dz - s * (1.0 + z * (1.0 - s)))[ok] <= (rel * s * (1.0 + np.abs(z)))[ok]).all()
    assert (y[1:] == 0.0).all() and abs(y[0] - h.sum()) <= 256 * 2.0**-23 * np.abs(h).sum()


def _chain(v, axis=0):
    """FP32 sums in order."""
    return np.add.accumulate(v.astype(np.float32), axis=axis, dtype=np.float32).take(-1, axis=axis)


@pytest.mark.parametrize("batch", [1, 33, 64, 65, 200, 1000])
def test_bias_sums_in_row_order(env, batch):
    """The bias gradients are sums in the order of the rows, 64 at a time, then
    the partial sums in order.  With b = 0 and W2 = W3 = 1 every activation is
    0, silu' = 1/2, and W4 = (1, ..) on one output gives dz3 = dy / 2 and
    dz2 = bf16(dz3) / 2, exactly: the sums can be formed again bit by bit."""
    rt, torch, tr = env
    say("bias sums batch=%d" % batch)
    w4 = np.zeros((6, 256))
    w4[np.arange(256) % 6, np.arange(256)] = 1.0
    pt, pb = _plain_net(torch, W2=np.eye(256), W3=np.eye(256), W4=w4)
    rng = np.random.default_rng(batch)
    dy = (rng.normal(size=(1, batch, 6)) * 2.0 ** rng.integers(-12, 12, (1, batch, 6))).astype(np.float32)
    work = tr.mlp_work(1, batch)
    tr.mlp_fwd(pb, pt, torch.zeros((1, batch, 6), device="cuda"), work)
    parts = mlp.split(tr.mlp_bwd(pb, pt, torch.tensor(dy, device="cuda"), work).cpu().numpy()[0])
    dz3 = 0.5 * dy[0][:, np.arange(256) % 6]
    dz2 = 0.5 * mlp.bf16_round(dz3).astype(np.float32)
    for got, dz in ((parts[5], dz3), (parts[3], dz2)):
        ref = _chain(np.stack([_chain(dz[r:r + 64]) for r in range(0, batch, 64)]))
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("batch", [193, 256, 264, 1000, 1024])
def test_weight_gradient_order(env, batch):
    """The weight gradients of the 256x256 layers run through the batch in one
    chain of 32-row products, or, for batches of whole 128 rows, in four
    quarters added as (q0 + q2) + (q1 + q3).  One row of each 32 carries a power
    of two (h2 = 64 where b2 = 64), among them a large one and its negative, next
    to which the others vanish: every sum is exact or keeps the large one."""
    rt, torch, tr = env
    say("weight gradient order batch=%d" % batch)
    pt, pb = _plain_net(torch, b2=64.0, W4=np.eye(6, 1) * np.ones(256))
    ns = (batch + 31) // 32
    ones = np.ones(ns, np.float32)
    ones[[ns // 4, ns // 2]] = 2.0**40, -2.0**40
    dy = np.zeros((1, batch, 6), np.float32)
    dy[0, ::32, 0] = ones
    work = tr.mlp_work(1, batch)
    tr.mlp_fwd(pb, pt, torch.zeros((1, batch, 6), device="cuda"), work)
    g = mlp.split(tr.mlp_bwd(pb, pt, torch.tensor(dy, device="cuda"), work).cpu().numpy()[0])[4]
    v = 32.0 * ones  # dz3 h2 = (dy / 2) 64
    if batch % 128 == 0:
        q = [_chain(v[ns * k // 4:ns * (k + 1) // 4]) for k in range(4)]
        ref = np.float32(q[0] + q[2]) + np.float32(q[1] + q[3])
    else:
        ref = _chain(v)
    assert (g == ref).all(), (g[0, 0], ref)


@pytest.mark.parametrize("n,batch", [(3, 100), (2, 128)])
def test_training_loop_equals_its_steps(env, n, batch):
    """The training loop across a border of its groups of 16 steps, against the
    same steps made one by one: the same bits."""
    rt, torch, tr = env
    say("training loop n_nets=%d batch=%d" % (n, batch))
    kappa, scale = np.linspace(0.4, 2.5, n).astype(np.float32), np.full(n, 0.3, np.float32)
    steps, lr, warmup, seed = 18, 2e-3, 200, 5
    state = []
    for _ in range(2):
        p, pt, pb = _params(torch, n)
        state.append([pt, pb, torch.zeros_like(pt), torch.zeros_like(pt)])
    log, _ = tr.surrogate_train(kappa, scale, *state[0], batch, steps, seed=seed, lr=lr, warmup=warmup, log_every=1)
    pt, pb, m, v = state[1]
    work = tr.mlp_work(n, batch)
    for step in range(1, steps + 1):
        if step % 16 == 1:
            X, Y, _ = tr.surrogate_gen(kappa, scale, 16 * batch, 0.01, mode=4, seed=seed + 1000003 * ((step - 1) // 16 + 1))
        j = (step - 1) % 16
        x, t = X[:, j::16].contiguous(), Y[:, j::16].contiguous()
        dy, part = tr.mse_grad(tr.mlp_fwd(pb, pt, x, work), t, batch)
        g = tr.mlp_bwd(pb, pt, dy, work)
        tr.adamw(pt, pb, m, v, g, float(np.float32(lr) * np.float32(step) / np.float32(warmup)), step)
        assert torch.equal(log[step - 1], part), step
    for a, b in zip(*state):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", [100, 16384, 16385, 400000])
def test_mse_summation_order(env, n):
    """Each of a block's 256 chains adds its squares in order, then the chains
    are added in halves.  With 12-bit differences the squares are exact, and the
    partial sums can be formed again bit by bit."""
    rt, torch, tr = env
    say("mse summation order n=%d" % n)
    rng = np.random.default_rng(n)
    d = (rng.integers(-4095, 4096, n) * 2.0 ** rng.integers(-20, 0, n)).astype(np.float32)
    _, part = tr.mse_grad(torch.tensor(d, device="cuda"), torch.zeros(n, device="cuda"), 7)
    sq = np.zeros(-(-n // 16384) * 16384, np.float32)
    sq[:n] = d * d
    s = _chain(sq.reshape(-1, 64, 256))
    while s.shape[1] > 1:
        s = s[:, :s.shape[1] // 2] + s[:, s.shape[1] // 2:]
    assert np.array_equal(part.cpu().numpy(), s[:, 0])


def test_grouped_forward_after_other_calls(env):
    """A long grouped call on one stream, another entry point and then a grouped
    call with other networks on a second stream: the second call waits for the
    first, whose networks it would overwrite."""
    rt, torch, tr = env
    say("grouped forward, other calls between")
    rng = np.random.default_rng(9)
    (_, pa, wa), (_, pb, wb) = _params(torch, 8), _params(torch, 8, scale=0.5)
    xa = torch.tensor(rng.normal(size=(800000, 6)).astype(np.float32), device="cuda")
    xb = xa[:640].contiguous()
    ra, rb = [100000] * 8, [80] * 8
    alone = tr.mlp_fwd_grouped(wa, pa, xa, ra).clone(), tr.mlp_fwd_grouped(wb, pb, xb, rb).clone()
    torch.cuda.synchronize()
    s0, s1 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(s0):
            ya = tr.mlp_fwd_grouped(wa, pa, xa, ra)
        with torch.cuda.stream(s1):
            tr.surrogate_gen([1.0], [0.3], 64, 0.01)
            yb = tr.mlp_fwd_grouped(wb, pb, xb, rb)
        torch.cuda.synchronize()
        assert torch.equal(ya, alone[0]) and torch.equal(yb, alone[1])


def test_grouped_forward_refuses_capture(env):
    """A graph would keep the address of the context's buffer."""
    rt, torch, tr = env
    say("grouped forward under capture")
    _, pt, pb = _params(torch, 2)
    x = torch.zeros((100, 6), device="cuda")
    ref = tr.mlp_fwd_grouped(pb, pt, x, [50, 50]).clone()
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        x + 1.0
        with pytest.raises(rt.RtError, match="captured"):
            tr.mlp_fwd_grouped(pb, pt, x, [50, 50])
    assert torch.equal(tr.mlp_fwd_grouped(pb, pt, x, [50, 50]), ref)


@pytest.mark.parametrize("batch", [3, 64, 66])
def test_many_small_networks(env, batch):
    """More networks than the workspace holds re-laid weights for, of one tile
    (which need none) and of two: the same as the networks by themselves, at a few
    hundred KB a network."""
    rt, torch, tr = env
    n = 515
    say("mlp n_nets=%d batch=%d" % (n, batch))
    assert rt._lib.rt_mlp_work_bytes(1, 1) < 1.0e6
    assert rt._lib.rt_mlp_work_bytes(4096, 1) < 1.3e9
    rng = np.random.default_rng(3)
    pt = torch.tensor(rng.normal(0.0, 0.06, (n, mlp.N_PARAMS)).astype(np.float32), device="cuda")
    pb = pt.to(torch.bfloat16)
    x = torch.tensor(rng.normal(size=(n, batch, 6)).astype(np.float32), device="cuda")
    dy = torch.tensor(rng.normal(size=(n, batch, 6)).astype(np.float32), device="cuda")
    work = tr.mlp_work(n, batch)
    y = tr.mlp_fwd(pb, pt, x, work)
    g = tr.mlp_bwd(pb, pt, dy, work)
    for a, b in ((0, 3), (254, 259), (510, 515)):
        w1 = tr.mlp_work(b - a, batch)
        assert torch.equal(tr.mlp_fwd(pb[a:b], pt[a:b], x[a:b], w1), y[a:b])
        assert torch.equal(tr.mlp_bwd(pb[a:b], pt[a:b], dy[a:b], w1), g[a:b])
