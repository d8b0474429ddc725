"""GPU parity of the front end: int8 quantisation, per-row length policy, and the
whole device pipeline fp32 -> int8 -> lengths -> SC GEMM against the oracle's.

Quantised integers, scales and lengths are integer (or exactly reproduced fp32)
decisions taken in fp32 on both sides: compared bit for bit."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _note(msg):
    print("[gpu-case] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32922_amd as scg
    scg.load()
    return torch.device("cuda:0")


def _t(x, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to(dev)


def test_quantize_rows_and_tensor(dev, oracle_mod):
    import paper_2609_32922_amd as scg
    rng = np.random.default_rng(3)
    X = rng.standard_normal((2, 150, 777)).astype(np.float32)
    X[:, :, 5] *= 30
    X[0, 7] = 0.0
    X[1, :, 100] = np.float32(1.5)        # ties after scaling are possible
    _note("quantize rows")
    Q, s, m = scg.quantize(_t(X, dev), per_tensor=False, want_rowmax=True)
    Q, s, m = Q.cpu().numpy(), s.cpu().numpy(), m.cpu().numpy()
    for b in range(2):
        Qr, sr, mr = oracle_mod.quantize_rows_fp32(X[b])
        assert np.array_equal(Q[b], Qr) and np.array_equal(s[b], sr) and np.array_equal(m[b], mr)
    _note("quantize tensor")
    Q, s, m = scg.quantize(_t(X, dev), per_tensor=True, want_rowmax=True)
    Q, s = Q.cpu().numpy(), s.cpu().numpy()
    for b in range(2):
        Qr, sr = oracle_mod.quantize_tensor_fp32(X[b])
        assert np.array_equal(Q[b], Qr) and np.array_equal(s[b], sr)


def test_quantize_full_size_against_host_quantiser(dev, oracle_mod):
    import paper_2609_32922_amd as scg
    rng = np.random.default_rng(1)
    X = rng.standard_normal((6304, 768)).astype(np.float32)
    X[:, rng.choice(768, 6, replace=False)] *= np.float32(20.0)
    _note("quantize 6304x768")
    Q, s, _ = scg.quantize(_t(X, dev))
    Q, s = Q.cpu().numpy(), s.cpu().numpy()
    Qh, sh = W.quantize_rows(X)
    assert np.array_equal(Q, Qh) and np.array_equal(s, sh)
    rows = [0, 1, 2, 4000, 6303]
    Qr, sr, _ = oracle_mod.quantize_rows_fp32(X[rows])
    assert np.array_equal(Q[rows], Qr) and np.array_equal(s[rows], sr)


def test_mp_lengths(dev, oracle_mod):
    import paper_2609_32922_amd as scg
    rng = np.random.default_rng(4)
    g = rng.gamma(2.0, 1.0, (3, 1001)).astype(np.float32)
    g[2] = np.float32(0.5)                # constant metric: shortest everywhere
    for tau, ladder in [([0.6, 0.3, 0.1], [192, 96, 48, 24]), ([], [77]),
                        ([0.5], [512, 8]), ([1.0, 0.0], [300, 200, 100])]:
        _note("mp_lengths %s %s" % (tau, ladder))
        L = scg.mp_lengths(_t(g, dev), tau, ladder).cpu().numpy()
        for b in range(3):
            assert np.array_equal(L[b], oracle_mod.mp_lengths_fp32(g[b], tau, ladder))


def test_mp_lengths_rejects_bad_ladders(dev):
    import torch
    import paper_2609_32922_amd as scg
    g = torch.ones(10, device=dev)
    for tau, ladder in [([0.5], [64, 64]), ([0.2, 0.5], [3, 2, 1]), ([1.5], [9, 3]), ([0.5], [9, -1])]:
        with pytest.raises(scg.ScError):
            scg.mp_lengths(g, tau, ladder)


def test_device_pipeline_end_to_end(dev, oracle_mod):
    """fp32 activations and weights -> device int8 + scales + row metric -> device
    lengths -> SC GEMM with the device length vector, against the oracle pipeline."""
    import torch
    import paper_2609_32922_amd as scg
    rng = np.random.default_rng(5)
    X = rng.standard_normal((300, 200)).astype(np.float32)
    X[:, 3] *= 12
    Wt = (rng.standard_normal((260, 200)) * 0.02).astype(np.float32)
    tau, ladder = [0.5, 0.25, 0.1], [160, 96, 48, 24]
    for pol in (0, 1):
        _note("pipeline polarity %d" % pol)
        qX, sX, mX = scg.quantize(_t(X, dev), want_rowmax=True)
        qW, sW, _ = scg.quantize(_t(Wt, dev), per_tensor=True)
        L = scg.mp_lengths(mX, tau, ladder)
        out, cnt = scg.gemm(qX, sX, qW, sW, L, L_max=160, polarity=pol, seed=11, want_counts=True,
                            check_status=True)
        torch.cuda.synchronize()
        oq, osx, om = oracle_mod.quantize_rows_fp32(X)
        ow, osw = oracle_mod.quantize_tensor_fp32(Wt)
        oL = oracle_mod.mp_lengths_fp32(om, tau, ladder)
        assert np.array_equal(L.cpu().numpy(), oL)
        c_ref, o_ref = oracle_mod.sc_gemm(oq, ow, osx, osw, oL, 160, pol, 11)
        assert np.array_equal(cnt.cpu().numpy(), c_ref)
        o = out.cpu().numpy().astype(np.float64)
        nz = o_ref != 0
        assert np.all(o[~nz] == 0)
        assert np.max(np.abs(o[nz] - o_ref[nz]) / np.abs(o_ref[nz])) <= 1e-6


def test_device_pipeline_with_threshold_table(dev, oracle_mod):
    """The policy of Sec. 4.4 with its calibrated-threshold table: per layer the table gives
    (thresholds, ladder) for the operator's timestep and layer bucket (or the operator-level
    fallback); the device turns the row metric into lengths, which drive the SC GEMM."""
    import os

    import torch
    import paper_2609_32922_amd as scg
    from paper_2609_32922_amd.thresholds import ThresholdTable, mp_lengths_from_table
    table = ThresholdTable.load(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden",
                                             "thresholds_synthetic.json"))
    rng = np.random.default_rng(6)
    X = rng.laplace(0.0, 1.0, (260, 120)).astype(np.float32)
    Wt = (rng.standard_normal((300, 120)) * 0.02).astype(np.float32)
    for op, t, layer, want in [("mlp_fc1", 3, 27, "bucket"), ("mlp_fc1", 40, 0, "operator"),
                               ("mlp_fc2", 12, 22, "bucket")]:
        _note("table pipeline %s t=%d layer=%d" % (op, t, layer))
        qX, sX, mX = scg.quantize(_t(X, dev), want_rowmax=True)
        qW, sW, _ = scg.quantize(_t(Wt, dev), per_tensor=True)
        L, thr = mp_lengths_from_table(mX, table, op, t, layer)
        assert thr.source == want
        L_max = thr.ladder[0]
        out, cnt = scg.gemm(qX, sX, qW, sW, L, L_max=L_max, polarity=1, seed=13, want_counts=True,
                            check_status=True)
        torch.cuda.synchronize()
        oq, osx, om = oracle_mod.quantize_rows_fp32(X)
        ow, osw = oracle_mod.quantize_tensor_fp32(Wt)
        oL = oracle_mod.mp_lengths_fp32(om, thr.tau, thr.ladder)
        assert np.array_equal(L.cpu().numpy(), oL)
        assert len(set(oL.tolist())) > 1
        c_ref, o_ref = oracle_mod.sc_gemm(oq, ow, osx, osw, oL, L_max, 1, 13)
        assert np.array_equal(cnt.cpu().numpy(), c_ref)
        o = out.cpu().numpy().astype(np.float64)
        nz = o_ref != 0
        assert np.all(o[~nz] == 0)
        assert np.max(np.abs(o[nz] - o_ref[nz]) / np.abs(o_ref[nz])) <= 1e-6


@pytest.mark.parametrize("K", [1, 3, 4, 255, 256, 257, 768, 769, 1280, 1284, 2047, 2048, 2052, 5000])
def test_quantize_row_lengths_and_ties(dev, oracle_mod, K):
    """Every register-held row length and the block per longer row, aligned and not (K, and rows of
    a wider matrix from an odd column on), at quotients on and beside the halves, where the
    product with the reciprocal may not decide, and with scales at both ends of fp32."""
    import torch
    import paper_2609_32922_amd as scg
    rng = np.random.default_rng(K)
    rows = 9
    X = rng.standard_normal((rows, K)).astype(np.float32)
    for i, top in enumerate((127.0, 1.0, 3.0e38, 1.3e-36, 2e-43, 0.0)):
        # quotients k / 2 of the scale top / 127, nudged by up to 2 ulps
        s = np.float32(top) / np.float32(127)
        h = (rng.integers(-254, 255, K) * np.float32(0.5)).astype(np.float32) * s
        h = np.where(rng.random(K) < 0.5, np.nextafter(h, np.float32(0)), h).astype(np.float32)
        h[rng.integers(K)] = np.float32(top)
        X[i] = np.clip(h, -np.float32(top), np.float32(top))
    _note("quantize K=%d" % K)
    for per_tensor in (False, True):
        Q, s, m = scg.quantize(_t(X, dev), per_tensor=per_tensor, want_rowmax=True)
        ref = oracle_mod.quantize_tensor_fp32(X) if per_tensor else oracle_mod.quantize_rows_fp32(X)
        assert np.array_equal(Q.cpu().numpy(), ref[0]) and np.array_equal(s.cpu().numpy(), ref[1])
    # rows inside wider matrices, from a column that is no multiple of 4 on: single elements
    wide = torch.zeros((rows, K + 11), device=dev)
    wide[:, 5:5 + K] = _t(X, dev)
    Qw = torch.full((rows, K + 7), 55, dtype=torch.int8, device=dev)
    sw = torch.empty(rows, device=dev)
    rc = scg.sc_quantize(1, rows, K, wide.data_ptr() + 5 * 4, K + 11, 0, 0, Qw.data_ptr() + 3, K + 7, 0, sw.data_ptr(), 0,
                         rows, int(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    ref = oracle_mod.quantize_rows_fp32(X)
    Qw = Qw.cpu().numpy()
    assert np.array_equal(Qw[:, 3:3 + K], ref[0]) and np.array_equal(sw.cpu().numpy(), ref[1])
    assert (Qw[:, :3] == 55).all() and (Qw[:, 3 + K:] == 55).all()


@pytest.mark.parametrize("M", [1, 1023, 1024, 1025, 20481, 40000])
def test_mp_lengths_many_blocks(dev, oracle_mod, M):
    import paper_2609_32922_amd as scg
    g = np.random.default_rng(M).gamma(2.0, 1.0, (2, M)).astype(np.float32)
    tau, ladder = [0.5, 0.25, 0.1], [256, 128, 64, 32]
    _note("mp lengths M=%d" % M)
    L = scg.mp_lengths(_t(g, dev), tau, ladder).cpu().numpy()
    for b in range(2):
        assert np.array_equal(L[b], oracle_mod.mp_lengths_fp32(g[b], tau, ladder))


@pytest.mark.parametrize("batch,M", [(3, 40000), (2000, 2500)])
def test_mp_lengths_over_the_metric(dev, oracle_mod, batch, M):
    """Lengths written over the metrics they come from: every metric of an entry is read before the
    entry's first length is written (also where an entry's blocks would not all run at once)."""
    import torch
    import paper_2609_32922_amd as scg
    g = np.random.default_rng(M).gamma(2.0, 1.0, (batch, M)).astype(np.float32)
    g[:, 0], g[:, -1] = 50.0, 0.0
    tau, ladder = [0.5, 0.25, 0.1], [256, 128, 64, 32]
    buf = _t(g, dev)
    _note("mp lengths over the metric, %d x %d" % (batch, M))
    rc = scg.sc_mp_lengths(batch, M, buf.data_ptr(), M, tau, ladder, buf.data_ptr(), M,
                           int(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    L = buf.cpu().numpy().view(np.int32)
    for b in range(0, batch, 1 + batch // 100):
        assert np.array_equal(L[b], oracle_mod.mp_lengths_fp32(g[b], tau, ladder))


@pytest.mark.parametrize("shape", [(5, 48), (1, 5, 48), (3, 4, 16)])
def test_binding_ranks_and_current_stream(dev, oracle_mod, shape):
    """Outputs have the rank of their input, own contiguous memory, and the launches go to the
    current stream or the given one: the same values on the default stream, on a current side
    stream and on a passed side stream."""
    import torch
    import paper_2609_32922_amd as scg
    g = torch.Generator(device="cpu").manual_seed(11)
    x = torch.randn(shape, generator=g).to(dev)
    tau, ladder = [0.5, 0.25, 0.1], [64, 40, 24, 12]
    B = torch.randint(-127, 128, (7, shape[-1]), dtype=torch.int8, generator=g).to(dev)
    sB = torch.full((7,), 0.02, device=dev)

    def call(stream):
        q, s, m = scg.quantize(x, want_rowmax=True, stream=stream)
        L = scg.mp_lengths(m, tau, ladder, stream=stream)
        out, counts = scg.gemm(q, s, B, sB, L, L_max=64, seed=3, want_counts=True, stream=stream)
        return q, s, m, L, out, counts

    _note("binding shape=%s" % (shape,))
    side = torch.cuda.Stream()
    want = call(None)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        current = call(None)
    torch.cuda.synchronize()
    given = call(side)
    torch.cuda.synchronize()
    shapes = [shape, shape[:-1], shape[:-1], shape[:-1], shape[:-1] + (7,), shape[:-1] + (7,)]
    for w, c, v, sh in zip(want, current, given, shapes):
        assert tuple(w.shape) == tuple(sh) and w.is_contiguous()
        assert torch.equal(w, c) and torch.equal(w, v)
    A = x.cpu().numpy().reshape(-1, shape[-1])
    absmax = np.abs(A).max(axis=1)
    assert np.array_equal(want[2].cpu().numpy().reshape(-1), absmax)
