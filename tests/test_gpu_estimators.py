"""LogLog and PCSA on the pool (the pool serves them too: the text after
Alg. 5, Sec. 5), HIP path vs oracle.  PCSA runs bit for bit after every
advance (direct and deferred scans); estimates within the HyperLogLog path's
bar: FP64 epilogues that differ only in the last bit of exp2/pow, so E_s to
1e-13 relative and the FP32 result to 1e-6 relative plus a floor for the
cancellation in (m E_s - g E_m)/(m - g)."""
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
    oracle.lib()
    return oracle


def _close(V, O, sk, osk, hosts, kind):
    hd = V.to_device_u32(hosts)
    out, raw = sk.estimate_kind(hd, kind, with_raw=True)
    out, raw = out.cpu().numpy(), raw.cpu().numpy()
    code = {"loglog": O.LOGLOG, "pcsa": O.PCSA}[kind]
    ref, ref_raw = osk.estimate_kind(hosts, code, with_raw=True)
    np.testing.assert_allclose(raw, ref_raw, rtol=1e-13, atol=0)
    m, g = float(osk.m), float(osk.g)
    floor = 1e-12 * (m * np.abs(ref_raw) + g * ref_raw.max()) / (m - g)
    bad = np.abs(out.astype(np.float64) - ref) > 1e-6 * np.abs(ref) + floor + 1e-6 * m * g / (m - g)
    assert not bad.any(), (kind, out[bad][:5], ref[bad][:5])


@pytest.mark.parametrize("m", [50021, (1 << 22) + 77])  # direct scans; deferred scans
def test_pcsa_and_loglog_match_oracle(V, O, m):
    g, k, seed = 128, 3, 51
    rng = np.random.default_rng(m % 997)
    aips = rng.integers(0, 2**32, 1500, dtype=np.uint64).astype(np.uint32)
    sk = V.Sketch(m, g, k, seed, "small")
    sk.enable_pcsa(True)
    with pytest.raises(V.VbdrError):  # no runs before an advance
        sk.estimate_kind(V.to_device_u32(aips[:4]), "pcsa")
    osk = O.Sketch(m, g, k, seed, O.GSMALL)
    hosts = np.concatenate([aips[:400], rng.integers(0, 2**32, 50, dtype=np.uint64).astype(np.uint32)])
    for t in range(5):
        n = 0 if t == 2 else int(rng.integers(1 << 16, 1 << 18))
        pairs = np.stack([aips[rng.integers(0, len(aips), n)],
                          rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)], 1).astype(np.uint32)
        if n:
            sk.scan_slice(V.to_device_u32(pairs.reshape(-1)))
        osk.scan(pairs)
        sk.advance_slice()
        osk.advance()
        assert np.array_equal(sk.pcsa_registers(), osk.pcsa_registers()), t
        for kind in ("loglog", "pcsa"):
            _close(V, O, sk, osk, hosts, kind)
    # the HyperLogLog kind is the plain estimate
    hd = V.to_device_u32(hosts)
    assert torch.equal(sk.estimate_kind(hd, "hll"), sk.estimate(hd))


def test_loglog_on_fast_layout_and_pcsa_refused(V, O):
    m, g, k, seed = 30011, 64, 2, 3
    rng = np.random.default_rng(5)
    aips = rng.integers(0, 2**32, 300, dtype=np.uint64).astype(np.uint32)
    sk = V.Sketch(m, g, k, seed, "fast")
    osk = O.Sketch(m, g, k, seed, O.GFAST)
    pairs = np.stack([aips[rng.integers(0, 300, 50000)],
                      rng.integers(0, 2**32, 50000, dtype=np.uint64).astype(np.uint32)], 1).astype(np.uint32)
    sk.scan_slice(V.to_device_u32(pairs.reshape(-1)))
    osk.scan(pairs)
    sk.advance_slice()
    osk.advance()
    _close(V, O, sk, osk, aips, "loglog")
    with pytest.raises(V.VbdrError):
        sk.enable_pcsa(True)
    with pytest.raises(V.VbdrError):
        sk.estimate_kind(V.to_device_u32(aips), "pcsa")


def test_failed_pcsa_allocation_leaves_sketch_whole(V):
    """An out-of-memory failure while enabling PCSA runs (either of its two
    allocations) returns VBDR_ENOMEM and leaves the sketch as it was: the
    LDS-tiled estimate's workspaces stay allocated and give the same
    estimates, PCSA stays off, and enabling it again afterwards works."""
    m, g, k = 1 << 24, 1024, 4
    rng = np.random.default_rng(77)
    aips = rng.integers(0, 2**32, 2000, dtype=np.uint64).astype(np.uint32)
    sk = V.Sketch(m, g, k, 3, "small")
    assert sk.info().est_tiled == 1
    n = 1 << 20
    pairs = np.stack([aips[rng.integers(0, len(aips), n)],
                      rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)], 1).astype(np.uint32)
    sk.scan_slice(V.to_device_u32(pairs.reshape(-1)))
    sk.advance_slice()
    hd = V.to_device_u32(aips)
    before = sk.estimate(hd)
    bytes0 = sk.info().state_bytes
    try:
        for after in (0, 1):  # the run array, then the pool sum
            V.fail_allocation_after(after)
            with pytest.raises(V.VbdrError) as e:
                sk.enable_pcsa(True)
            assert e.value.code == -2
            V.fail_allocation_after(-1)
            assert sk.info().state_bytes == bytes0 and sk.info().est_tiled == 1
            assert torch.equal(sk.estimate(hd), before)
            with pytest.raises(V.VbdrError) as e:
                sk.estimate_kind(hd, "pcsa")
            assert e.value.code == -4
    finally:
        V.fail_allocation_after(-1)
    sk.enable_pcsa(True)
    sk.advance_slice()
    assert sk.estimate_kind(hd, "pcsa").shape == (len(aips),)
    sk.close()


@pytest.mark.parametrize("m,g", [(5000, 4), (70_001, 128), (100_000, 32768), ((1 << 22) + 1, 64), ((1 << 23) + 9, 2048),
                                 ((1 << 24) + 1, 256), ((1 << 25) + 5, 1024)])
def test_sum_routes(V, m, g):
    """The sums of LogLog and PCSA by a wave a host, 16 lanes a host and in pool
    ranges: LogLog's raw E_s is the one of estimate_ex's histograms, up to the
    rounding of its constant, and of either kind a host's results do not depend
    on the hosts it is estimated with (a few take the direct gathers)."""
    rng = np.random.default_rng(g + 1)
    sk = V.Sketch(m, g, 3, 21, "small")
    sk.enable_pcsa(True)
    for _ in range(2):
        sk.scan_slice(V.to_device_u32(rng.integers(0, 2**32, min(m, 1 << 24) * 2, dtype=np.uint64).astype(np.uint32)))
        sk.advance_slice()
    hosts = rng.integers(0, 2**32, 33_001, dtype=np.uint64).astype(np.uint32)
    hd = V.to_device_u32(hosts)
    few = min(len(hosts), max(1, ((1 << 20) - 1) // g))  # fewer gathers than ranges need
    _, _, hist = sk.estimate_ex(hd[:few])
    S = (hist.double().cpu() * torch.arange(33, dtype=torch.float64)).sum(1)
    lit = (g * torch.exp2(S / g)).numpy()
    for kind in ("pcsa", "loglog"):
        out, raw = sk.estimate_kind(hd, kind, with_raw=True)
        if kind == "loglog":
            ratio = raw[:few].cpu().numpy() / lit
            assert np.ptp(ratio) <= 1e-13 * ratio[0]
        for n in (1, 3, 17, 255, 16_385):
            a, b = (0, n) if n <= few else (len(hosts) - n, len(hosts))
            o, r = sk.estimate_kind(hd[a:b].contiguous(), kind, with_raw=True)
            assert torch.equal(o, out[a:b]) and torch.equal(r, raw[a:b]), (kind, n)


@pytest.mark.parametrize("m,g,nh", [((1 << 24) + 1, 256, 30_001), ((1 << 25) + 5, 1024, 9_000), ((1 << 23) + 5, 2048, 9_000),
                                    ((1 << 23) + 5, 4096, 9_000)])
def test_sums_share_nothing_between_streams(V, m, g, nh):
    """LogLog, PCSA and HyperLogLog estimates of one sketch on three streams at
    once, in pool ranges (different hosts each): the results of one after the other."""
    rng = np.random.default_rng(g + 2)
    sk = V.Sketch(m, g, 3, 21, "small")
    sk.enable_pcsa(True)
    sk.scan_slice(V.to_device_u32(rng.integers(0, 2**32, m // 2 * 2, dtype=np.uint64).astype(np.uint32)))
    sk.advance_slice()
    hosts = [V.to_device_u32(rng.integers(0, 2**32, nh, dtype=np.uint64).astype(np.uint32)) for _ in range(3)]
    kinds = ("loglog", "pcsa", "hll")
    alone = [sk.estimate_kind(h, k) for h, k in zip(hosts, kinds)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in kinds]
    for _ in range(10):
        outs = []
        for h, k, s in zip(hosts, kinds, streams):
            with torch.cuda.stream(s):
                outs.append(sk.estimate_kind(h, k))
        torch.cuda.synchronize()
        for a, o, k in zip(alone, outs, kinds):
            assert torch.equal(a, o), k


def test_est_blocks_per_cu_bounds_every_estimate(V):
    """est_blocks_per_cu = 1 gives the plain, LogLog, PCSA and feature kernels one
    workgroup per CU, directly and in ranges: the same bits, and more time than the
    default takes (the same, within a few percent, where the bound has no effect)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    for m in (3_000_000, 12_000_000):
        sk = V.Sketch(m, 64, 3, 21, "small")
        sk.enable_pcsa(True)
        sk.scan_slice(torch.randint(-2**31, 2**31, (2 * m,), dtype=torch.int64, device="cuda", generator=gen).to(torch.int32))
        sk.advance_slice()
        hosts = torch.randint(-2**31, 2**31, (400_000,), dtype=torch.int64, device="cuda", generator=gen).to(torch.int32)
        calls = {"hll": lambda: sk.estimate(hosts), "loglog": lambda: sk.estimate_kind(hosts, "loglog"),
                 "pcsa": lambda: sk.estimate_kind(hosts, "pcsa"), "features": lambda: sk.features(hosts[:32_000])}
        for name, f in calls.items():
            us, outs = [], []
            for b in (64, 1):
                sk.set_tuning(est_blocks_per_cu=b)
                outs.append(f())
                best = float("inf")
                for _ in range(10):
                    x, y = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    x.record()
                    f()
                    y.record()
                    y.synchronize()
                    best = min(best, x.elapsed_time(y) * 1e3)
                us.append(best)
            assert torch.equal(outs[0], outs[1]), (m, name)
            assert name == "features" or us[1] > 1.15 * us[0], (m, name, us)  # half of its time is not the histograms


@pytest.mark.parametrize("m,g", [(300, 16), (5003, 64), (1 << 16, 1024), ((1 << 16) + 1, 256), (200_001, 2048),
                                 (100_000, 16384)])
@pytest.mark.parametrize("share", [1 / 33, 1 / 31, 1 / 17, 1 / 15, 1 / 5, 1 / 3, 1.0])
def test_pools_of_large_registers(V, m, g, share):
    """Shares of registers of 15 and more around the ones from which the gathers read
    bytes and not nibbles (from L2, from LDS, for histograms): plain estimates
    and features are estimate_ex's, LogLog sums its histograms' up to the
    rounding of the constant."""
    rng = np.random.default_rng(g)
    sk = V.Sketch(m, g, 3, 21, "small")
    reg = rng.integers(0, min(sk.L, 14) + 1, m).astype(np.uint8)
    wide = rng.permutation(m)[: int(m * share)]
    reg[wide] = rng.integers(min(15, sk.L), sk.L + 1, len(wide))
    sk.load_state({"dr": np.full((m, sk.L), 255, np.uint8), "reg": reg,
                   "hist": np.bincount(reg, minlength=33).astype(np.uint64), "t": 1})
    hosts = V.to_device_u32(rng.integers(0, 2**32, 17_001, dtype=np.uint64).astype(np.uint32))
    ref, _, hist = sk.estimate_ex(hosts)
    for n in (1, 5, 1025, 5000, 17_001):
        h = hosts[:n].contiguous()
        assert torch.equal(sk.estimate(h), ref[:n]), n
        assert torch.equal(sk.features(h)[:, :33], (hist[:n].double() / g).float()), n
        raw = sk.estimate_kind(h, "loglog", with_raw=True)[1].cpu().numpy()
        S = (hist[:n].double().cpu() * torch.arange(33, dtype=torch.float64)).sum(1)
        ratio = raw / (g * torch.exp2(S / g)).numpy()
        assert np.ptp(ratio) <= 1e-13 * ratio[0], n


def test_large_registers_cost_no_second_gather(V):
    """Estimates of a pool whose registers are 15 and more against one of as many
    small registers: about the same time (1.8 to 2 times while every gather of a
    nibble of 15 was followed by one of its byte)."""
    m, g = 40_000, 1024
    rng = np.random.default_rng(1)
    hosts = V.to_device_u32(rng.integers(0, 2**32, 100_000, dtype=np.uint64).astype(np.uint32))
    us = {}
    for lo in (2, 15):
        sk = V.Sketch(m, g, 3, 21, "small")
        reg = rng.integers(lo, lo + 4, m).astype(np.uint8)
        sk.load_state({"dr": np.full((m, sk.L), 255, np.uint8), "reg": reg,
                       "hist": np.bincount(reg, minlength=33).astype(np.uint64), "t": 1})
        best = float("inf")
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sk.estimate_kind(hosts, "loglog")
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3)
        us[lo] = best
    assert us[15] < 1.4 * us[2], us
