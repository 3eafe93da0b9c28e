"""Learned estimator on the GPU vs the FP64 reference (oracle/mlp_ref.py).

Features are bit-exact (same FP64 divisions rounded once to FP32).  The
network output y = ln(1 + n) agrees within 1e-4 |y| + 2e-3: the GPU
accumulates in FP32 on the matrix cores where the reference uses FP64, and a
first-layer activation sitting on a bf16 rounding boundary may round the
other way (one bf16 ulp, 2^-8 relative, times a weight).  Gradients of one
batch agree within 1e-3 relative (FP32 accumulation over the batch and the
network), the Adam update to 1e-6 absolute.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_13132_amd import vbdr
    vbdr.lib()
    return vbdr


@pytest.fixture(scope="module")
def O():
    from oracle import oracle
    return oracle


@pytest.fixture(scope="module")
def M():
    from oracle import mlp_ref
    return mlp_ref


def _build(V, O, m, g, k, seed, layout="fast", n_slices=4, n_pairs=60000, n_aip=600):
    rng = np.random.default_rng(seed)
    aips = rng.integers(0, 2**32, n_aip, dtype=np.uint64).astype(np.uint32)
    sk = V.Sketch(m, g, k, seed, layout)
    osk = O.Sketch(m, g, k, seed, O.GFAST if layout == "fast" else O.GSMALL)
    for _ in range(n_slices):
        sizes = rng.zipf(1.3, n_aip).clip(1, 5000)
        a = np.repeat(aips, sizes)
        b = rng.integers(0, 2**32, len(a), dtype=np.uint64).astype(np.uint32)
        pairs = np.stack([a, b], 1)[rng.permutation(len(a))][:n_pairs].astype(np.uint32)
        sk.scan_slice(V.to_device_u32(pairs.reshape(-1)))
        osk.scan(pairs)
        sk.advance_slice()
        osk.advance()
    hosts = np.concatenate([aips, rng.integers(0, 2**32, 37, dtype=np.uint64).astype(np.uint32)])
    return sk, osk, hosts


def _random_params(M, seed):
    p = M.init_params(seed)
    p[M.N_PARAMS - 1] = 5.0  # output bias: ln(1 + n) around e^5
    return p


@pytest.mark.parametrize("m,g,layout", [(20011, 64, "fast"), ((1 << 22) + 5, 256, "small")])
def test_features_bit_exact(V, O, M, m, g, layout):
    sk, osk, hosts = _build(V, O, m, g, 3, 7, layout)
    f = sk.features(V.to_device_u32(hosts)).cpu().numpy()
    _, hist = osk.estimate(hosts, with_hist=True)
    ref = M.features(hist, osk.state()["hist"], g, m).astype(np.float32)
    assert np.array_equal(f, ref)


@pytest.mark.parametrize("m,g,layout", [(20011, 64, "fast"), (50021, 256, "small"), ((1 << 22) + 5, 256, "fast")])
def test_learned_inference_matches_fp64(V, O, M, m, g, layout):
    sk, osk, hosts = _build(V, O, m, g, 3, 11, layout)
    params = _random_params(M, 3)
    mlp = V.MLP(params)
    hd = V.to_device_u32(hosts)
    out, fb = sk.estimate_learned(mlp, hd, with_fallback=True)
    out, fb = out.cpu().numpy(), fb.cpu().numpy()
    assert not fb.any()
    _, hist = osk.estimate(hosts, with_hist=True)
    feats = M.features(hist, osk.state()["hist"], g, m)
    y = M.infer(params, feats)
    y_gpu = np.log1p(out.astype(np.float64))
    ok = np.abs(y_gpu - y) <= 1e-4 * np.abs(y) + 2e-3
    ok |= (out == 0) & (np.expm1(y) <= 1e-3)  # clamped at 0
    assert ok.all(), (y_gpu[~ok][:5], y[~ok][:5])


def test_learned_fallback_is_the_plain_estimate(V, O, M):
    sk, osk, hosts = _build(V, O, 30011, 128, 4, 5)
    params = _random_params(M, 4)
    lo = np.full(67, -1e30, np.float32)
    hi = np.full(67, 1e30, np.float32)
    hi[66] = -100.0  # ln(g/m) outside the envelope: every host falls back
    mlp = V.MLP(params, lo, hi)
    hd = V.to_device_u32(hosts)
    out, fb = sk.estimate_learned(mlp, hd, with_fallback=True)
    assert fb.cpu().numpy().all()
    assert torch.equal(out, sk.estimate(hd))
    wide = V.MLP(params, lo, np.full(67, 1e30, np.float32))
    _, fb2 = sk.estimate_learned(wide, hd, with_fallback=True)
    assert not fb2.cpu().numpy().any()


@pytest.mark.parametrize("m,layout", [(30011, "fast"), ((1 << 22) + 5, "small")])
def test_learned_plain_above_keeps_large_counts(V, O, M, m, layout):
    """With a threshold, hosts whose plain estimate reaches it keep the plain
    estimate bit for bit (flag 2) and the others keep the network's output
    (flag 0); no threshold (inf) gives the network's output everywhere.  The
    second case takes the partitioned histogram path of large pools."""
    sk, osk, hosts = _build(V, O, m, 128, 4, 5, layout)
    params = _random_params(M, 4)
    hd = V.to_device_u32(hosts)
    plain = sk.estimate(hd)
    out0, fb0 = sk.estimate_learned(V.MLP(params), hd, with_fallback=True)
    assert not fb0.any()
    thr = float(torch.quantile(plain.double(), 0.6))
    cut = V.MLP(params, plain_above=thr)
    out1, fb1 = sk.estimate_learned(cut, hd, with_fallback=True)
    big = plain >= thr
    assert 0 < int(big.sum()) < len(hosts)
    assert torch.equal(fb1 == 2, big) and not (fb1 == 1).any()
    assert torch.equal(out1[big], plain[big]) and torch.equal(out1[~big], out0[~big])
    with pytest.raises(V.VbdrError):
        cut.set_plain_above(0.0)
    cut.set_plain_above(float("inf"))
    out2, fb2 = sk.estimate_learned(cut, hd, with_fallback=True)
    assert torch.equal(out2, out0) and not fb2.any()


def test_train_gradient_matches_fp64(V, M):
    rng = np.random.default_rng(0)
    params = _random_params(M, 9)
    feats = rng.uniform(0, 1, (300, 67)).astype(np.float32)
    feats[:, 66] = -6.0
    targets = rng.uniform(0, 9, 300).astype(np.float32)
    tr = V.Trainer(params, 1e-3)
    g, loss = tr.grad(torch.from_numpy(feats).cuda(), torch.from_numpy(targets).cuda())
    ref_loss, ref_g = M.loss_and_grad(params.astype(np.float64), feats.astype(np.float64), targets.astype(np.float64))
    g = g.cpu().numpy().astype(np.float64)
    assert abs(float(loss.cpu()[0]) - ref_loss) <= 1e-4 * ref_loss
    scale = np.abs(ref_g).max()
    np.testing.assert_allclose(g, ref_g, rtol=1e-3, atol=1e-4 * scale)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 8193])
def test_train_gradient_batch_edges(V, M, n):
    """Batches at the edges of the gradient kernel's tiles (16 samples), of a
    workgroup's four tiles and of its grid, against float64; grads_out is
    added to.  fp32 sums of n terms: the tolerance of the test above."""
    rng = np.random.default_rng(n)
    params = _random_params(M, 9)
    feats = rng.uniform(0, 1, (n, 67)).astype(np.float32)
    targets = rng.uniform(0, 9, n).astype(np.float32)
    tr = V.Trainer(params, 1e-3)
    g, loss = tr.grad(torch.from_numpy(feats).cuda(), torch.from_numpy(targets).cuda())
    ref_loss, ref_g = M.loss_and_grad(params.astype(np.float64), feats.astype(np.float64), targets.astype(np.float64))
    assert abs(float(loss.cpu()[0]) - ref_loss) <= 1e-4 * ref_loss
    np.testing.assert_allclose(g.cpu().numpy().astype(np.float64), ref_g, rtol=1e-3, atol=1e-4 * np.abs(ref_g).max())


def test_train_step_is_adam(V, M):
    rng = np.random.default_rng(1)
    params = _random_params(M, 10)
    feats = rng.uniform(0, 1, (128, 67)).astype(np.float32)
    targets = rng.uniform(0, 9, 128).astype(np.float32)
    tr = V.Trainer(params, 1e-3)
    fd, td = torch.from_numpy(feats).cuda(), torch.from_numpy(targets).cuda()
    g, _ = tr.grad(fd, td)
    tr.step(fd, td)
    ref, _, _ = M.adam_step(params.astype(np.float64), np.zeros(M.N_PARAMS), np.zeros(M.N_PARAMS),
                            g.cpu().numpy().astype(np.float64), 1, lr=1e-3)
    np.testing.assert_allclose(tr.params(), ref, rtol=0, atol=1e-6)


def test_training_reduces_loss(V, M):
    rng = np.random.default_rng(2)
    feats = rng.uniform(0, 1, (4096, 67)).astype(np.float32)
    targets = (3 * feats[:, 0] + np.sin(4 * feats[:, 1]) + 2).astype(np.float32)
    fd, td = torch.from_numpy(feats).cuda(), torch.from_numpy(targets).cuda()
    tr = V.Trainer(M.init_params(1), 3e-3)
    first = float(tr.grad(fd, td)[1].cpu()[0])
    for _ in range(300):
        tr.step(fd, td)
    last = float(tr.grad(fd, td)[1].cpu()[0])
    assert last < 0.05 * first


@pytest.mark.parametrize("m,g", [(300, 2), (5000, 16), (70_001, 2048), (70_001, 4096), (1 << 17, 8192), (100_000, 16384),
                                 ((1 << 22) + 1, 64), ((1 << 23) + 9, 256), ((1 << 24) + 1, 512), ((1 << 25) + 5, 128)])
def test_histogram_routes(V, M, m, g):
    """Histograms counted in registers (16 and 64 lanes a host, up to 128
    registers a lane), with LDS atomics and in 1, 2 and 4 pool ranges: the
    features are the ones of estimate_ex's histograms, and a network that
    rejects every host returns the plain estimates.  Small pools hold planted
    registers, a tenth of them 15 and more, and most others one value."""
    rng = np.random.default_rng(g)
    sk = V.Sketch(m, g, 3, 21, "small")
    if m < 1 << 20:
        reg = np.full(m, 3, np.uint8)
        other = rng.random(m) < 0.3
        reg[other] = rng.integers(0, sk.L + 1, int(other.sum()))
        hist = np.bincount(reg, minlength=33).astype(np.uint64)
        sk.load_state({"dr": np.full((m, sk.L), 255, np.uint8), "reg": reg, "hist": hist, "t": 1})
    else:
        sk.scan_slice(V.to_device_u32(rng.integers(0, 2**32, m, dtype=np.uint64).astype(np.uint32)[: m // 2 * 2]))
        sk.advance_slice()
    hosts = rng.integers(0, 2**32, 33_001, dtype=np.uint64).astype(np.uint32)
    plain, _, hist = sk.estimate_ex(V.to_device_u32(hosts))
    pool = torch.from_numpy(sk.registers()[1].astype(np.float64) / m).float().cuda()
    want = (hist.double() / g).float()
    mlp = V.MLP(_random_params(M, 3), np.full(67, 2.0, np.float32), np.full(67, 1.0, np.float32))
    for n in (1, 3, 17, 1025, 4_097, 8_193, 32_768, 33_001):
        hd = V.to_device_u32(hosts[:n])
        f = sk.features(hd)
        assert torch.equal(f[:, :33], want[:n]) and torch.equal(f[:, 33:66], pool.expand(n, 33)), n
        assert torch.equal(f[:, 66], torch.full((n,), float(np.float32(np.log(g / m))), device="cuda")), n
        est, fb = sk.estimate_learned(mlp, hd, with_fallback=True)
        assert bool((fb == 1).all()) and torch.equal(est, plain[:n]), n


@pytest.mark.parametrize("m,g", [(1 << 22, 2048), ((1 << 22) + 5, 8192), (1 << 23, 4096), ((1 << 25) + 5, 2048)])
def test_learned_hosts_do_not_depend_on_their_list(V, M, m, g):
    """Few hosts of large g go through the histogram pass, more in one launch: a
    host's learned estimate and flag are the same bits either way."""
    rng = np.random.default_rng(g)
    sk = V.Sketch(m, g, 3, 21, "small")
    sk.scan_slice(V.to_device_u32(rng.integers(0, 2**32, m // 2 * 2, dtype=np.uint64).astype(np.uint32)))
    sk.advance_slice()
    hosts = rng.integers(0, 2**32, 3_000, dtype=np.uint64).astype(np.uint32)
    mlp = V.MLP(_random_params(M, 3))
    out, fb = sk.estimate_learned(mlp, V.to_device_u32(hosts), with_fallback=True)
    for n in (1, 15, 17, 1023, 1024, 1025):
        o, f = sk.estimate_learned(mlp, V.to_device_u32(hosts[:n]), with_fallback=True)
        assert torch.equal(o, out[:n]) and torch.equal(f, fb[:n]), n


def test_few_learned_hosts_cost_few(V, M):
    """64 hosts of g = 8192 on a pool that fills the L2s against 2000: half of the
    time (more than all of it while four workgroups gathered them)."""
    m, g = 1 << 23, 8192
    sk = V.Sketch(m, g, 3, 21, "small")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    sk.scan_slice(torch.randint(-2**31, 2**31, (2 * m,), dtype=torch.int64, device="cuda", generator=gen).to(torch.int32))
    sk.advance_slice()
    hosts = torch.randint(-2**31, 2**31, (2000,), dtype=torch.int64, device="cuda", generator=gen).to(torch.int32)
    mlp = V.MLP(_random_params(M, 3))
    us = {}
    for n in (64, 2000):
        h, best = hosts[:n].contiguous(), float("inf")
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sk.estimate_learned(mlp, h)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        us[n] = best
    assert us[64] < 0.75 * us[2000], us
