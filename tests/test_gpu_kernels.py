"""Parity of each HIP kernel with the CPU oracle on identical seeded inputs, element by
element, through the C ABI.  Integer work (codes, zero sets) must be bit-exact; binary32
state is expected bit-exact too (both sides follow the same arithmetic contract) and is
asserted within the stated tolerance of 1e-5 max relative error, with exactness reported."""
import numpy as np
import pytest
import torch

import oracle
from paper_2208_05631_amd import synth

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2208_05631_amd as qa
    from gpu_util import DEV, GpuState, dev, gpu_quantize_pack, host, quantizer_parity, sampled_tiles, ulp_distance, workspace

RTOL = 1e-5


def make_grad(kind, M, d, seed):
    rng = np.random.default_rng(seed)
    if kind == "gauss":
        g = rng.standard_normal((M, d)) * 1e-2 + rng.standard_normal((M, 1)) * 3e-3
    elif kind == "laplace_sparse":
        g = rng.laplace(0, 1e-3, (M, d)) * (rng.random((M, d)) < 0.05)
    elif kind == "student":
        g = rng.standard_t(3, (M, d)) * 1e-2 * (rng.random((M, d)) < 0.1)
    elif kind == "mixed_scale":
        g = rng.standard_normal((M, d)) * (10.0 ** rng.integers(-6, 3, (M, 1)))
    elif kind == "zeros":
        g = np.zeros((M, d))
    else:
        raise ValueError(kind)
    return g.astype(np.float32)


def assert_close(a, b, what):
    assert a.shape == b.shape, what
    if np.array_equal(a, b):
        return
    denom = np.maximum(np.abs(b), 1e-30)
    err = np.max(np.abs(a.astype(np.float64) - b) / denom)
    assert err <= RTOL, f"{what}: max rel err {err}"


# ------------------------------------------------------------------ quantize + pack

QP_CASES = [
    # d, M, bucket
    (1, 1, 0), (15, 2, 0), (16, 1, 64), (17, 3, 64), (1000, 4, 0), (1000, 2, 256),
    (4096, 2, 4096), (4097, 2, 4096), (10000, 3, 1024), (10000, 3, 2048), (12289, 2, 512),
    (70001, 2, 4096), (70001, 2, 8192), (70001, 2, 65536), (70001, 3, 0), (300000, 2, 128),
]


@pytest.mark.parametrize("d,M,bucket", QP_CASES)
@pytest.mark.parametrize("kind", ["gauss", "laplace_sparse"])
def test_quantize_pack_matches_oracle(d, M, bucket, kind):
    g = make_grad(kind, M, d, seed=d * 7 + M)
    oc, osc, oth = oracle.quantize_pack(g, bucket=bucket)
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    # bit-identical, or (about once in 2^29 sums) a threshold / scale one ulp off with codes that
    # are exact for the GPU's own threshold
    assert quantizer_parity(g, bucket, codes, scales, th) <= 1


_MID = []


def mid_size_gradient():
    """4 workers x 2^26 coordinates, 30 % non-zero, Laplace(0, 1e-3) magnitudes; drawn on the
    device by the seeded input generator and copied to the host once."""
    if not _MID:
        _MID.append(np.stack([host(synth.grad_laplace_sparse(1 << 26, m, 1, seed=2024, keep=0.3,
                                                             device=DEV)) for m in range(4)]))
    return _MID[0]


@pytest.mark.parametrize("bucket", [4096, 256, 0])
def test_every_threshold_and_scale_at_a_mid_size(bucket):
    """All buckets of a 2^26-coordinate message from each of 4 workers (2 x 65 536 sums per worker
    at bucket 4096, 16 times that at 256): thresholds, scales and codes against the oracle.  The
    two sides add the same binary64 terms in different orders, so a rounded sum may differ in its
    last binary32 bit about once in 2^29 sums: the count of such buckets is reported, each must
    lie within one ulp, and the codes must be exact for the GPU's own thresholds."""
    g = mid_size_gradient()
    M, d = g.shape
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    off = quantizer_parity(g, bucket, codes, scales, th)
    print(f"bucket {bucket}: {off} of {M * L.n_buckets} (worker, bucket) pairs not bit-identical")
    assert off <= 4


@pytest.mark.parametrize("bucket", [4096, 1024, 0])
def test_quantizer_on_magnitudes_spread_over_many_binades(bucket):
    """Partial sums of a bucket are exact in binary64 only while the magnitudes span few enough
    binades (span + log2 n + 24 <= 53); beyond that each side rounds its own partial sums.  With
    magnitudes over 60 binades the results may therefore differ, but only in the last bit."""
    d, M = 50000, 3
    rng = np.random.default_rng(77)
    g = (rng.standard_normal((M, d)) * np.exp2(rng.integers(-40, 20, (M, d)))).astype(np.float32)
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    off = quantizer_parity(g, bucket, codes, scales, th)
    print(f"bucket {bucket}: {off} of {M * L.n_buckets} (worker, bucket) pairs not bit-identical")


def test_quantize_pack_strides_and_untouched_padding():
    d, M, b = 5000, 3, 1024
    g = make_grad("gauss", M, d, 5)
    codes, scales, th, L = gpu_quantize_pack(g, b, code_stride=400, scale_stride=9, g_stride=5008)
    oc, osc, oth = oracle.quantize_pack(g, bucket=b, code_stride=400, scale_stride=9)
    W, nb = L.words, L.n_buckets
    assert np.array_equal(codes[:, :W], oc[:, :W]) and np.array_equal(scales[:, :nb], osc[:, :nb])
    assert np.all(codes[:, W:] == 0xFFFFFFFF) and np.all(scales[:, nb:] == -7.0)   # not written


@pytest.mark.parametrize("bucket", [0, 256, 4096, 16384])
def test_quantize_pack_with_given_thresholds(bucket):
    d, M = 40000, 2
    g = make_grad("gauss", M, d, 11)
    nb = oracle.n_buckets(d, bucket)
    rng = np.random.default_rng(1)
    thr = (rng.random((M, nb)) * 1e-2).astype(np.float32)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket, thresholds=thr)
    codes, scales, th, L = gpu_quantize_pack(g, bucket, thresholds=thr)
    assert np.array_equal(codes, oc) and np.array_equal(scales[:, :nb], osc[:, :nb])
    assert np.array_equal(th[:, :nb], thr)                                          # left as given


@pytest.mark.parametrize("bucket", [0, 64, 4096])
def test_quantize_degenerate_inputs(bucket):
    d, M = 9000, 2
    g = make_grad("zeros", M, d, 0)
    g[1, 100] = np.nan            # poisons its bucket only: threshold NaN, codes 0, scale 0
    g[1, 8000:] = 0.5
    oc, osc, oth = oracle.quantize_pack(g, bucket=bucket)
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    nb = L.n_buckets
    assert np.array_equal(codes, oc)
    assert np.array_equal(scales[:, :nb], osc[:, :nb])
    assert np.array_equal(np.isnan(th[:, :nb]), np.isnan(oth[:, :nb]))
    assert np.array_equal(np.nan_to_num(th[:, :nb]), np.nan_to_num(oth[:, :nb]))
    assert not codes[0].any() and not scales[0, :nb].any()


# ------------------------------------------------------------------ aggregate

@pytest.mark.parametrize("d,M,bucket", [(1, 1, 0), (1000, 4, 0), (5000, 3, 64), (70001, 6, 4096),
                                        (70001, 64, 4096), (33333, 7, 16384), (20000, 33, 1024),
                                        # complete chunks of 16 and of 8 workers whose last tile ends
                                        # inside a 16-byte group of a row of code words
                                        (9000, 48, 4096), (8192 + 16 * 5 + 3, 8, 4096), (70001, 24, 0),
                                        (4096 + 16 * 62 + 1, 32, 8192)])
def test_aggregate_matches_oracle(d, M, bucket):
    g = make_grad("mixed_scale" if M <= 7 else "gauss", M, d, seed=M + d)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    L = qa.Layout.make(d, M, bucket)
    out = torch.full((d,), 9.0, dtype=torch.float32, device=DEV)
    qa.qa_aggregate_unpack(L, dev(oc.view(np.int32)), dev(osc), out)
    torch.cuda.synchronize()
    assert np.array_equal(host(out), oracle.aggregate(oc, osc, d, bucket=bucket))


@pytest.mark.parametrize("d,M,bucket", [(70001, 64, 4096), (50000, 130, 8192), (9000, 70, 0),
                                        (20000, 5, 4096)])
def test_aggregate_with_widely_spread_scales_takes_the_ordered_path(d, M, bucket):
    """Scales spanning > 29 - log2(M) binades inside a bucket: the sum is no longer exact in
    binary64, so only worker order reproduces the oracle's rounding."""
    rng = np.random.default_rng(M)
    g = rng.standard_normal((M, d)).astype(np.float32) * (2.0 ** rng.integers(-40, 40, (M, 1))).astype(np.float32)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    L = qa.Layout.make(d, M, bucket)
    out = torch.zeros(d, dtype=torch.float32, device=DEV)
    qa.qa_aggregate_unpack(L, dev(oc.view(np.int32)), dev(osc), out)
    torch.cuda.synchronize()
    ref = oracle.aggregate(oc, osc, d, bucket=bucket)
    assert np.array_equal(host(out), ref)
    # half the buckets get narrow spans again: both paths inside one launch
    nb = L.n_buckets
    osc2 = osc.copy()
    osc2[:, : max(1, nb // 2)] = (1e-3 * (1 + rng.random((M, max(1, nb // 2))))).astype(np.float32)
    qa.qa_aggregate_unpack(L, dev(oc.view(np.int32)), dev(osc2), out)
    torch.cuda.synchronize()
    assert np.array_equal(host(out), oracle.aggregate(oc, osc2, d, bucket=bucket))


def test_aggregate_with_nonfinite_scale_matches_oracle():
    d, M, b = 10000, 8, 4096
    g = make_grad("gauss", M, d, 9)
    oc, osc, _ = oracle.quantize_pack(g, bucket=b)
    osc[3, 1] = np.inf                      # inf * 0 = NaN, inf * +-1 = +-inf: bucket 1 is poisoned
    out = torch.zeros(d, dtype=torch.float32, device=DEV)
    qa.qa_aggregate_unpack(qa.Layout.make(d, M, b), dev(oc.view(np.int32)), dev(osc), out)
    torch.cuda.synchronize()
    ref = oracle.aggregate(oc, osc, d, bucket=b)
    assert not np.isfinite(ref[4096:8192]).any() and np.isfinite(ref[:4096]).all()
    assert np.array_equal(host(out), ref, equal_nan=True)


def test_aggregate_reads_reserved_pattern_as_zero_and_ignores_tail_bits():
    d, M = 40, 2
    rng = np.random.default_rng(3)
    words = rng.integers(0, 2 ** 32, (M, 3), dtype=np.uint64).astype(np.uint32)   # all 4 patterns
    scales = np.array([[0.5], [0.25]], np.float32)
    for bucket in (0, 64):                 # table-driven sum / worker-ordered sum
        L = qa.Layout.make(d, M, bucket)
        out = torch.zeros(d, dtype=torch.float32, device=DEV)
        qa.qa_aggregate_unpack(L, dev(words.view(np.int32)), dev(scales), out)
        torch.cuda.synchronize()
        assert np.array_equal(host(out), oracle.aggregate(words, scales, d, bucket=bucket))


# ------------------------------------------------------------------ fused steps

STEP_CASES = [
    # d, M, bucket, requant
    (1, 1, 0, 0), (1000, 4, 0, 0), (1000, 4, 0, 2), (4096, 8, 4096, 0), (4097, 8, 4096, 1),
    (10000, 3, 64, 1), (10000, 5, 256, 1), (10000, 16, 1024, 1), (10000, 2, 2048, 1),
    (70001, 64, 4096, 0), (70001, 32, 4096, 1), (70001, 6, 4096, 2), (70001, 4, 16384, 1),
    (70001, 4, 16384, 0), (300001, 8, 4096, 0), (50001, 130, 4096, 0), (50001, 67, 4096, 1),
    (20000, 128, 4096, 1),
    # chunking of the table-driven kernel: 3 chunks of 8, 3 chunks of 16, guarded chunks (20 = 16 + 4, 12)
    (9000, 24, 4096, 0), (9000, 48, 4096, 1), (9000, 20, 0, 0), (9000, 12, 4096, 2), (9000, 40, 8192, 0),
    # buckets smaller than the tile without in-kernel second quantization: per-thread scales
    (10000, 3, 64, 0), (10000, 9, 256, 0), (70001, 16, 1024, 0), (70001, 64, 2048, 2), (4100, 8, 512, 2),
    # the largest worker count the layout accepts, and a large odd one
    (5000, 4096, 4096, 0), (3000, 1001, 0, 2),
    # second quantization over buckets that span tiles: few workers (the average is formed from the
    # messages in every pass) with chunks of 16, 8, 4 and guarded chunks; many workers (the average
    # is written to the workspace once)
    (70001, 16, 0, 2), (70001, 8, 8192, 1), (70001, 3, 0, 2), (70001, 13, 16384, 1), (9000, 16, 64, 2),
    (70001, 24, 0, 2), (70001, 20, 16384, 1),
    # ... and where that second quantization is a one-pass one although it is not formed in the
    # step kernel (single tile, messages with smaller buckets), or spans "several" tiles of one
    (3000, 4, 64, 2), (4096, 8, 1024, 2), (50, 3, 8192, 1),
]


@pytest.mark.parametrize("d,M,bucket,requant", STEP_CASES)
def test_fused_steps_match_oracle_over_several_steps(d, M, bucket, requant):
    eta, lam, delta = 0.1, 2e-4, 1e-8
    rng = np.random.default_rng(d + M)
    x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
    ox, oG, oz = x0.copy(), np.zeros(d, np.float32), np.zeros(d, np.float32)
    L = qa.Layout.make(d, M, bucket)
    st = None
    T = 6
    for t in range(1, T + 1):
        g = make_grad("gauss" if t % 2 else "laplace_sparse", M, d, seed=1000 * t + d)
        oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
        if st is None:
            st = GpuState(L, oc, osc, ox, oG, oz)
        else:
            st.codes.copy_(dev(oc.view(np.int32)))
            st.scales.copy_(dev(osc))
        if t % 3 == 0:                       # QRDA steps overwrite x from (z, G, t)
            oracle.step_qrda(oc, osc, d, bucket, ox, oG, oz, t, eta, lam, delta, requant)
            st.qrda(t, eta, lam, delta, requant)
        else:                                # QCMD steps keep z current
            oracle.step_qcmd(oc, osc, d, bucket, ox, oG, oz, eta, lam, delta, requant)
            st.qcmd(eta, lam, delta, requant, track_z=True)
        x, G, z = st.get()
        assert np.array_equal(x == 0, ox == 0), f"zero set differs at step {t}"
        assert_close(G, oG, f"G step {t}")
        assert_close(z, oz, f"z step {t}")
        assert_close(x, ox, f"x step {t}")
    assert np.array_equal(x, ox) and np.array_equal(G, oG) and np.array_equal(z, oz), \
        "within tolerance but not bit-identical"


@pytest.mark.parametrize("method", ["qcmd", "qcmd_z", "qrda"])
@pytest.mark.parametrize("requant", [0, 1])
def test_update_with_state_and_scalars_at_the_ends_of_the_exponent_range(method, requant):
    """For tiles whose scales lie in a safe exponent window the kernel takes short forms of the
    correctly rounded sqrt and division, and falls back to the full forms for any group of lanes
    whose accumulator (or, for QRDA, |z| - t*lambda) leaves the window.  State planted with tiny,
    huge, zero, negative-zero and non-finite values next to ordinary ones, and hyper-parameters
    inside and outside the window, must all give the oracle's bits."""
    d, M, bucket = 5 * 4096, 16, 4096
    rng = np.random.default_rng(404)
    g = make_grad("laplace_sparse", M, d, seed=5)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    L = qa.Layout.make(d, M, bucket)
    pool = np.array([0.0, -0.0, 1e-45, 1e-40, 3e-39, 1e-35, 1e-30, 1.2e-29, 1.3e-29, 1e-20, 1e-6, 1.0,
                     1e20, 8e37, 9e37, 3e38, np.inf, np.nan], np.float32)
    for case, (eta, lam, delta, t) in enumerate([(0.1, 2e-4, 1e-8, 3), (0.1, 0.0, 1e-8, 1),
                                                 (1e-20, 1e-3, 1e-8, 2), (0.1, 2e-4, 1e-30, 5),
                                                 (3e3, 1e-38, 1e10, 7), (0.1, 1e30, 1e-8, 4)]):
        x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
        G0 = (rng.random(d) * 1e-5).astype(np.float32)
        z0 = (rng.standard_normal(d) * 1e-3).astype(np.float32)
        where = rng.random(d) < 0.02                       # a few lanes per wave
        G0[where] = np.abs(rng.choice(pool, int(where.sum())))
        where = rng.random(d) < 0.02
        z0[where] = rng.choice(pool, int(where.sum())) * rng.choice([-1, 1], int(where.sum()))
        tl = np.float32(t) * np.float32(lam)
        where = rng.random(d) < 0.02                       # |z| - t*lambda just above / below zero
        z0[where] = (tl * (1 + rng.integers(-3, 4, int(where.sum())) * 2.0 ** -23)).astype(np.float32)
        where = rng.random(d) < 0.01
        x0[where] = rng.choice(pool, int(where.sum())) * rng.choice([-1, 1], int(where.sum()))
        ox, oG, oz = x0.copy(), G0.copy(), z0.copy()
        st = GpuState(L, oc, osc, x0, G0, z0)
        if method == "qrda":
            oracle.step_qrda(oc, osc, d, bucket, ox, oG, oz, t, eta, lam, delta, requant)
            st.qrda(t, eta, lam, delta, requant)
        else:
            tz = method == "qcmd_z"
            oracle.step_qcmd(oc, osc, d, bucket, ox, oG, oz if tz else None, eta, lam, delta, requant)
            st.qcmd(eta, lam, delta, requant, track_z=tz)
        x, G, z = st.get()
        for name, a, o in (("x", x, ox), ("G", G, oG), ("z", z, oz)):
            same = (a.view(np.uint32) == o.view(np.uint32)) | (np.isnan(a) & np.isnan(o))
            assert same.all(), (case, name, int((~same).sum()), a[~same][:4], o[~same][:4])


def test_qcmd_without_z_leaves_z_alone():
    d, M, b = 9000, 4, 4096
    g = make_grad("gauss", M, d, 77)
    oc, osc, _ = oracle.quantize_pack(g, bucket=b)
    ox, oG = np.zeros(d, np.float32), np.zeros(d, np.float32)
    z0 = np.full(d, 3.0, np.float32)
    st = GpuState(qa.Layout.make(d, M, b), oc, osc, ox, oG, z0)
    oracle.step_qcmd(oc, osc, d, b, ox, oG, None, 0.1, 1e-4, 1e-8)
    st.qcmd(0.1, 1e-4, 1e-8, 0, track_z=False)
    x, G, z = st.get()
    assert np.array_equal(x, ox) and np.array_equal(G, oG) and np.array_equal(z, z0)


def test_checkpoint_resume_is_bit_identical():
    """State is three tensors and t: T steps in one go == T/2, copy out, copy in, T/2."""
    d, M, b = 20000, 4, 4096
    L = qa.Layout.make(d, M, b)
    msgs = [oracle.quantize_pack(make_grad("gauss", M, d, 300 + t), bucket=b)[:2] for t in range(6)]
    zero = np.zeros(d, np.float32)

    def run(st, ts):
        for t in ts:
            st.codes.copy_(dev(msgs[t - 1][0].view(np.int32)))
            st.scales.copy_(dev(msgs[t - 1][1]))
            st.qrda(t, 0.1, 1e-4, 1e-8) if t % 2 == 0 else st.qcmd(0.1, 1e-4, 1e-8)
        return st.get()

    full = run(GpuState(L, msgs[0][0], msgs[0][1], zero, zero, zero), range(1, 7))
    half = run(GpuState(L, msgs[0][0], msgs[0][1], zero, zero, zero), range(1, 4))
    resumed = run(GpuState(L, msgs[0][0], msgs[0][1], *half), range(4, 7))
    for a, c in zip(full, resumed):
        assert np.array_equal(a, c)


# ------------------------------------------------------------------ local gradient

@pytest.mark.parametrize("d,B", [(1000, 64), (1003, 64), (4100, 13), (6144, 1), (257, 50)])
def test_local_grad_dense_matches_oracle(d, B):
    rng = np.random.default_rng(5)
    n = 512
    A = rng.standard_normal((n, d)).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    rows = rng.integers(0, n, B).astype(np.int32)
    x = (rng.standard_normal(d) * 0.05).astype(np.float32)
    og, ol = oracle.local_grad_dense(A, y, rows, x)
    L = qa.Layout.make(d, 1, 0)
    ws = workspace(qa.qa_workspace_bytes(L, qa.QA_OP_GRAD_DENSE))
    g = torch.full((d,), 5.0, dtype=torch.float32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    qa.qa_local_grad(qa.QA_DENSE, dev(A), None, None, n, d, dev(y), dev(rows), B, dev(x), g, loss, ws)
    torch.cuda.synchronize()
    gg = host(g)
    assert np.allclose(gg, og, rtol=1e-6, atol=1e-12)
    assert host(loss)[0] == pytest.approx(ol, rel=1e-6)
    print("dense grad bit-identical entries:", (gg == og).mean())
    assert (gg == og).mean() > 0.999


@pytest.mark.parametrize("d,B,M", [(1, 1, 1), (3, 65, 2), (5, 16, 3), (511, 64, 2), (513, 80, 2), (63, 1025, 1),
                                   (1023, 1040, 2), (257, 2049, 1), (12290, 64, 5)])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_local_grad_dense_at_any_alignment_and_batch_split(d, B, M, shift):
    """Matrix and x starting `shift` floats past a 16-byte boundary (and rows of odd length anywhere), batches
    around the shares of sixteen rows and the 1024 row ids staged at a time, ids outside the
    matrix (which add nothing), short and long rows."""
    rng = np.random.default_rng(d + B)
    n = 200
    A = rng.standard_normal((n, d)).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    x = (rng.standard_normal(d) * 0.1).astype(np.float32)
    rows = rng.integers(0, n, (M, B)).astype(np.int32)
    gs = (d + 3) // 4 * 4 + 4
    A_d = dev(np.concatenate([np.full(shift, np.nan, np.float32), A.reshape(-1)]))[shift:]
    x_d = dev(np.concatenate([np.full(shift, np.nan, np.float32), x]))[shift:]
    ws = workspace(qa.qa_workspace_bytes(qa.Layout.make(d, M, 0), qa.QA_OP_GRAD_DENSE))
    g = torch.full((M, gs), 5.0, dtype=torch.float32, device=DEV)
    loss = torch.zeros(M, dtype=torch.float32, device=DEV)
    ref = [oracle.local_grad_dense(A, y, rows[m], x) for m in range(M)]
    for with_bad in (False, True):
        ids = rows.copy()
        if with_bad and B > 16:                          # a row replaced by one outside: its term is missing
            ids[:, 7], ids[:, B - 1] = -1, n
            gone = [oracle.local_grad_dense(A, y, np.repeat(rows[m, [7, B - 1]], 1), x)[0] * (2.0 / B) for m in range(M)]
        qa.qa_local_grad_batched(qa.QA_DENSE, A_d, None, None, n, d, dev(y), dev(ids), B, M, x_d, g, gs, loss, ws)
        torch.cuda.synchronize()
        gg = host(g)
        R = np.stack([r[0] for r in ref])
        assert np.all(gg[:, d:] == 5.0)
        if with_bad and B > 16:
            # the reference less two terms, each rounded to binary32: 2^-23 of the larger operand
            assert np.allclose(gg[:, :d], R - np.stack(gone), rtol=1e-6, atol=4e-7 * np.abs(R).max())
        else:
            assert np.allclose(gg[:, :d], R, rtol=1e-6, atol=1e-30)
            assert np.allclose(host(loss), [r[1] for r in ref], rtol=1e-6)


# just below and above 2^27 components of different rows; short rows, few and many work-groups of columns
@pytest.mark.parametrize("d,B,M", [(300, 55925, 8), (4099, 8187, 4), (262147, 65, 8)])
@pytest.mark.parametrize("above", [False, True])
def test_local_grad_dense_around_the_line_of_streamed_batches(d, B, M, above):
    rng = np.random.default_rng(d)
    n, base = (1 << 27) // d + (1 if above else 0), 16   # the rows repeat every sixteen
    A = rng.standard_normal((base, d)).astype(np.float32)
    y = np.where(rng.random(base) < 0.5, -1.0, 1.0).astype(np.float32)
    x = (rng.standard_normal(d) * 0.01).astype(np.float32)
    rows = np.arange(M * B, dtype=np.int32).reshape(M, B) % n
    A_d, y_d = dev(A).repeat(-(-n // base), 1)[:n], dev(y).repeat(-(-n // base))[:n]
    gs = (d + 3) // 4 * 4
    ws = workspace(qa.qa_workspace_bytes(qa.Layout.make(d, M, 0), qa.QA_OP_GRAD_DENSE))
    g, loss = torch.full((M, gs), 5.0, dtype=torch.float32, device=DEV), torch.zeros(M, dtype=torch.float32, device=DEV)
    qa.qa_local_grad_batched(qa.QA_DENSE, A_d, None, None, n, d, y_d, dev(rows), B, M, dev(x), g, gs, loss, ws)
    torch.cuda.synchronize()
    for m in range(M):
        og, ol = oracle.local_grad_dense(A, y, rows[m] % base, x)
        # binary64 sums of terms up to coef * |A| <= 6 / B each, rounded to binary32 once
        assert np.all(np.abs(host(g)[m, :d] - og) <= np.spacing(np.abs(og)) + 6 * 2.0 ** -40)
        assert host(loss)[m] == pytest.approx(ol, rel=1e-6)


def _random_csr(rng, n, d, k):
    idx = np.stack([np.sort(rng.choice(d, k, replace=False)) for _ in range(n)]).astype(np.int32)
    vals = rng.standard_normal((n, k)).astype(np.float32)
    indptr = (np.arange(n + 1) * k).astype(np.int64)
    return vals.reshape(-1), indptr, idx.reshape(-1)


def test_local_grad_csr_matches_oracle():
    rng = np.random.default_rng(6)
    n, d, k, B = 300, 5000, 40, 128          # many column collisions -> atomics are exercised
    vals, indptr, idx = _random_csr(rng, n, d, k)
    idx = (idx % 200).astype(np.int32)       # hot columns (duplicates inside a row are summed too)
    y = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    rows = rng.integers(0, n, B).astype(np.int32)
    x = (rng.standard_normal(d) * 0.1).astype(np.float32)
    og, ol = oracle.local_grad_csr(vals, indptr, idx, d, y, rows, x)
    L = qa.Layout.make(d, 1, 0)
    ws = workspace(qa.qa_workspace_bytes(L, qa.QA_OP_GRAD_CSR))
    ws.fill_(0xAB)                            # contents on entry must not matter
    g = torch.full((d,), 5.0, dtype=torch.float32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    for _ in range(2):                        # second call reuses the dirty workspace
        qa.qa_local_grad(qa.QA_CSR, dev(vals), dev(indptr), dev(idx), n, d, dev(y), dev(rows), B,
                         dev(x), g, loss, ws)
    torch.cuda.synchronize()
    gg = host(g)
    assert np.array_equal(gg != 0, og != 0), "CSR indexing: non-zero set differs"
    assert np.allclose(gg, og, rtol=1e-6, atol=1e-12)
    assert host(loss)[0] == pytest.approx(ol, rel=1e-6)
    assert (gg == og).mean() > 0.999


@pytest.mark.parametrize("d,n,B,M,nnz", [(1, 9, 5, 1, 2), (40, 50, 384, 3, 30), (1024, 300, 70, 2, 40),
                                         (1025, 300, 17, 2, 40), (5003, 400, 300, 4, 150), (262145, 600, 130, 2, 70),
                                         (1 << 19, 300, 16, 3, 300), ((1 << 20) + 3, 500, 1100, 1, 60),
                                         ((1 << 21) + 1, 100, 33, 1, 50), (1 << 22, 64, 64, 1, 20),
                                         ((1 << 22) + 1, 64, 64, 1, 20),
                                         # no group, and about half of the groups, without room
                                         (1025, 300, 400, 2, 600), (900, 200, 300, 1, 330),
                                         # batches just within the rows that the form takes, and just beyond them
                                         (4099, 300, 750, 2, 100), (4099, 300, 820, 2, 100), (70000, 300, 1200, 1, 150),
                                         (200000, 300, 2000, 1, 60), (300000, 300, 2800, 1, 60), (1 << 20, 400, 8192, 1, 40),
                                         (1 << 21, 400, 16000, 1, 40), (1 << 21, 400, 17000, 1, 40)])
def test_local_grad_csr_across_the_column_ranges(d, n, B, M, nnz):
    """Lengths around every width of the column ranges and the last one that takes them, batches with more
    entries than the workspace has room for (read again from the rows), rows of different lengths (also
    empty ones), duplicate columns, columns outside the vector and row ids outside the matrix."""
    rng = np.random.default_rng(d + B)
    lens = rng.integers(0, 2 * nnz, n)
    lens[0] = 0
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(indptr[-1])
    idx = np.where(rng.random(total) < 0.5, rng.integers(0, d, total), rng.integers(0, max(1, d // 64), total))
    if total > 4:
        idx[:2] = [d - 1, 0]
    idx = idx.astype(np.int32)
    vals = rng.standard_normal(max(total, 1)).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    x = (rng.standard_normal(d) * 0.1).astype(np.float32)
    rows = rng.integers(0, n, (M, B)).astype(np.int32)
    rows[:, 0] = 0
    gs = (d + 3) // 4 * 4 + 8
    ws = workspace(qa.qa_workspace_bytes(qa.Layout.make(d, M, 0), qa.QA_OP_GRAD_CSR))
    ws.fill_(0xFF)
    g = torch.full((M, gs), 5.0, dtype=torch.float32, device=DEV)
    loss = torch.zeros(M, dtype=torch.float32, device=DEV)
    ip_d, y_d, x_d, v_d = dev(indptr), dev(y), dev(x), dev(vals)
    for bad in (False, True):
        ix, ids = idx.copy(), rows.copy()
        if bad and total > 4:                            # entries of row 0.. moved outside: they add nothing
            ix[::97] = np.where(np.arange(len(ix[::97])) % 2, -1, d).astype(np.int32)
        if bad:
            ids[:, -1] = n + 3
        qa.qa_local_grad_batched(qa.QA_CSR, v_d, ip_d, dev(ix), n, d, y_d, dev(ids), B, M, x_d, g, gs, loss, ws)
        torch.cuda.synchronize()
        gg, ll = host(g), host(loss)
        v2 = np.where((ix < 0) | (ix >= d), np.float32(0), vals[:total])
        i2 = np.where((ix < 0) | (ix >= d), 0, ix).astype(np.int32)
        assert np.all(gg[:, d:] == 5.0)
        for m in range(M):
            keep = ids[m] < n
            if not keep.any():
                continue
            og, ol = oracle.local_grad_csr(v2, indptr, i2, d, y, ids[m][keep], x)
            if keep.all():
                assert np.array_equal(gg[m, :d] != 0, og != 0)
                assert np.allclose(gg[m, :d], og, rtol=1e-6, atol=1e-30)
                assert ll[m] == pytest.approx(ol, rel=1e-6)
            else:                                        # the oracle divides by the rows kept: coefficients
                # rounded to binary32 after another division, 2^-23 each
                assert np.allclose(gg[m, :d], og * (keep.sum() / B), rtol=1e-5, atol=1e-6 * np.abs(og).max())


def test_local_grad_csr_with_2_to_the_32_entries_in_sixteen_rows():
    """Sixteen times the same row of 2^28 entries (columns repeat): as many entries as a 32-bit counter has
    values, which must not look like none.  All values equal, so that the gradient is known."""
    d, n, B = 300, 1 << 28, 16
    idx = torch.arange(n, device=DEV, dtype=torch.int32).remainder_(d)
    vals = torch.full((n,), 2.0 ** -20, dtype=torch.float32, device=DEV)
    x = dev(np.random.default_rng(1).standard_normal(d).astype(np.float32) * 0.01)
    L = qa.Layout.make(d, 1, 0)
    size, guard = qa.qa_workspace_bytes(L, qa.QA_OP_GRAD_CSR), 1 << 20
    ws = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    g, loss = torch.zeros(d, dtype=torch.float32, device=DEV), torch.zeros(1, dtype=torch.float32, device=DEV)
    qa.qa_local_grad(qa.QA_CSR, vals, dev(np.array([0, n], np.int64)), idx, 1, d, dev(np.ones(1, np.float32)),
                     dev(np.zeros(B, np.int32)), B, x, g, loss, ws[:size])
    torch.cuda.synchronize()
    assert bool((ws[size:] == 0xA5).all())
    per_column = np.bincount(np.arange(n % d), minlength=d) + n // d
    row = per_column * 2.0 ** -20
    p = np.float32(row @ host(x).astype(np.float64))
    coef = np.float32(-1.0 / (1.0 + np.exp(np.float64(p))) / B)
    # 2^32 / d additions in binary64 and the rounding of coef and g to binary32
    assert np.allclose(host(g), B * float(coef) * row, rtol=1e-6)
    assert host(loss)[0] == pytest.approx(np.log1p(np.exp(-np.float64(p))), rel=1e-6)


@pytest.mark.parametrize("csr,shape", [(False, (400, 3000, 30, 48, 5)), (True, (400, 3000, 30, 48, 5)),
                                       # large batches, heavy collisions on a few columns, a ragged last row group
                                       (True, (600, 5000, 30, 301, 7)), (True, (600, 1500, 20, 256, 8))])
def test_local_grad_batched_equals_per_worker_calls_and_oracle(csr, shape):
    rng = np.random.default_rng(8)
    n, d, k, B, M = shape
    y = np.where(rng.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    x = (rng.standard_normal(d) * 0.1).astype(np.float32)
    rows = rng.integers(0, n, (M, B)).astype(np.int32)
    if csr:
        vals, indptr, idx = _random_csr(rng, n, d, k)
        if B > 100:
            idx = np.where(rng.random(idx.size) < 0.6, idx % 37, idx).astype(np.int32)   # hot columns
        A_d, ip_d, ix_d = dev(vals), dev(indptr), dev(idx)
        ref = [oracle.local_grad_csr(vals, indptr, idx, d, y, rows[m], x) for m in range(M)]
        fmt, op = qa.QA_CSR, qa.QA_OP_GRAD_CSR
    else:
        A = rng.standard_normal((n, d)).astype(np.float32)
        A_d, ip_d, ix_d = dev(A), None, None
        ref = [oracle.local_grad_dense(A, y, rows[m], x) for m in range(M)]
        fmt, op = qa.QA_DENSE, qa.QA_OP_GRAD_DENSE
    gs = d + 8
    ws = workspace(qa.qa_workspace_bytes(qa.Layout.make(d, M, 0), op))
    g = torch.full((M, gs), 5.0, dtype=torch.float32, device=DEV)
    loss = torch.zeros(M, dtype=torch.float32, device=DEV)
    qa.qa_local_grad_batched(fmt, A_d, ip_d, ix_d, n, d, dev(y), dev(rows), B, M, dev(x), g, gs, loss, ws)
    torch.cuda.synchronize()
    gg, ll = host(g), host(loss)
    assert np.all(gg[:, d:] == 5.0)                      # padding between workers untouched
    for m in range(M):
        assert np.array_equal(gg[m, :d] != 0, ref[m][0] != 0)
        assert np.allclose(gg[m, :d], ref[m][0], rtol=1e-6, atol=1e-12)
        assert ll[m] == pytest.approx(ref[m][1], rel=1e-6)
    assert (gg[:, :d] == np.stack([r[0] for r in ref])).mean() > 0.999


# ------------------------------------------------------------------ stochastic ternary quantizer

@pytest.mark.parametrize("d,M,bucket", [(1, 1, 0), (1000, 3, 0), (4096, 2, 4096), (70001, 3, 4096),
                                        (70001, 2, 16384), (70001, 2, 0), (300001, 2, 4096),
                                        (70001, 2, 64), (12289, 3, 256), (70001, 2, 1024), (70001, 2, 2048),
                                        (100, 2, 512)])
def test_stochastic_quantizer_matches_oracle(d, M, bucket):
    g = make_grad("gauss" if d % 2 else "laplace_sparse", M, d, seed=d + 3)
    if d > 9000:
        g[0, 4096:8192] = 0.0                       # an all-zero tile: scale 0, nothing kept
    seed, step = 0x1234567811223344, 17
    oc, osc = oracle.quantize_pack_stochastic(g, bucket=bucket, seed=seed, step=step)
    L = qa.Layout.make(d, M, bucket)
    gs = ((d + 3) // 4) * 4
    gp = np.zeros((M, gs), np.float32); gp[:, :d] = g
    codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
    scales = torch.full((M, L.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack_stochastic(L, dev(gp), gs, codes, scales, seed, step)
    torch.cuda.synchronize()
    assert np.array_equal(host(scales)[:, :L.n_buckets], osc)
    assert np.array_equal(host(codes).view(np.uint32)[:, :L.words], oc)
    c2 = torch.zeros_like(codes)
    qa.qa_quantize_pack_stochastic(L, dev(gp), gs, c2, scales, seed, step + 1)
    torch.cuda.synchronize()
    assert d < 100 or not torch.equal(c2, codes)    # another step, other draws


# buckets of 2 .. 16 tiles are held in registers; 65537 components under one scale are the first that are not
@pytest.mark.parametrize("bucket,d", [(8192, 5 * 8192 - 7), (16384, 16384 + 4097), (32768, 2 * 32768 + 4096), (32768, 20481),
                                      (65536, 3 * 65536 - 4095), (65536, 40000), (0, 4097), (0, 12291), (0, 32769),
                                      (0, 65536), (0, 65537)])
def test_stochastic_quantizer_of_buckets_held_in_registers_matches_oracle(bucket, d):
    """Incomplete last tiles and buckets, buckets longer than the vector, a bucket of zeros, NaN."""
    rng = np.random.default_rng(d)
    M, seed, step = 3, 0xFEDCBA9876543210, 5
    g = rng.standard_normal((M, d)).astype(np.float32)
    g[0, :4096], g[1, d - 1], g[2, :65536] = 0, np.nan, 0
    oc, osc = oracle.quantize_pack_stochastic(g, bucket=bucket, seed=seed, step=step)
    L, gs = qa.Layout.make(d, M, bucket), (d + 3) // 4 * 4 + 4
    gp = np.full((M, gs), 9, np.float32)                  # padding belongs to nobody
    gp[:, :d] = g
    codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
    scales = torch.full((M, L.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack_stochastic(L, dev(gp), gs, codes, scales, seed, step)
    torch.cuda.synchronize()
    assert np.array_equal(host(scales)[:, :L.n_buckets], osc)
    assert np.array_equal(host(codes).view(np.uint32)[:, :L.words], oc)
    assert (host(codes)[:, L.words:] == -1).all() and (host(scales)[:, L.n_buckets:] == -7).all()


@pytest.mark.parametrize("bucket", [64, 256, 2048, 4096, 8192])
def test_stochastic_quantizer_at_the_ends_of_binary32(bucket):
    """Scales whose reciprocal is not a normal number (below 2^-126, above 2^126), around those ends, infinite."""
    rng = np.random.default_rng(bucket)
    ends = [2.0 ** -149, 1e-44, 1e-39, 2.0 ** -128, 2.0 ** -127, 2.0 ** -126, 1.5e-38, 1e-30, 1.0, 2.0 ** 125, 2.0 ** 126,
            1e38, 3.4e38, np.inf]
    parts = []
    for e in ends:
        v = np.exp2(rng.uniform(-12, 0, bucket)) * rng.choice([-1.0, 1.0], bucket)
        v *= 1.0 if e == np.inf else e
        v[bucket // 2] = e                              # the largest
        parts.append(v.astype(np.float32))
    g = np.stack([np.concatenate(parts), np.concatenate(parts[::-1])])
    d, M, seed, step = g.shape[1], 2, 0x0123456789ABCDEF, 3
    oc, osc = oracle.quantize_pack_stochastic(g, bucket=bucket, seed=seed, step=step)
    L = qa.Layout.make(d, M, bucket)
    codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
    scales = torch.full((M, L.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack_stochastic(L, dev(g), d, codes, scales, seed, step)
    torch.cuda.synchronize()
    assert np.array_equal(host(scales)[:, :L.n_buckets], osc)
    assert np.array_equal(host(codes).view(np.uint32)[:, :L.words], oc)


# ---- the server's call: messages in, q_t = Q(SynQ_t) out as a message ---------------------------

AGGQ_CASES = [
    # d, M, bucket, requant (1 = per bucket, 2 = one scale for the vector)
    (1, 1, 0, 2), (1000, 4, 0, 2), (4096, 8, 4096, 1), (4097, 8, 4096, 1), (70001, 16, 4096, 1),
    (70001, 20, 4096, 2), (10000, 3, 64, 1), (10000, 5, 256, 1), (70001, 6, 2048, 1),
    (70001, 4, 16384, 1), (70001, 4, 0, 2), (9000, 48, 4096, 1), (4100, 8, 512, 2),
    (70001, 16, 0, 2), (70001, 8, 8192, 1), (70001, 13, 0, 2), (70001, 24, 16384, 1),
    # one scale everywhere, up to 8 workers: three passes of the kernel that walks several tiles
    (70001, 8, 0, 2), (70001, 7, 0, 2), (4096 * 16400 + 5, 2, 0, 2), (4097, 1, 0, 2),
    # complete chunks of 16 and of 8 workers, one to four of them, rows ending inside a 16-byte group
    (70001, 32, 4096, 1), (70001, 64, 4096, 1), (9000, 24, 4096, 1), (8192 + 16 * 7 + 5, 40, 4096, 1),
]


@pytest.mark.parametrize("M", [3, 8, 24])
@pytest.mark.parametrize("spread", [30, 60, 100])
def test_one_scale_for_the_average_when_buckets_lie_far_apart(M, spread):
    """Messages with a scale per 4096-bucket whose magnitudes differ by up to 2^spread from bucket
    to bucket, and ONE scale for Q(SynQ): that scale is set by the largest buckets, so in most
    tiles q = +-s lies far outside the range of the tile's own scales (which is what decides
    whether the update may use the short forms of its division)."""
    d, bucket = 70001, 4096
    rng = np.random.default_rng(M * 1000 + spread)
    nb = (d + bucket - 1) // bucket
    g = make_grad("gauss", M, d, seed=M + spread)
    factor = np.exp2(rng.integers(-spread, spread // 3, nb)).astype(np.float32)
    g = g * np.repeat(factor, bucket)[:d][None, :]
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    L = qa.Layout.make(d, M, bucket)
    x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
    G0 = (rng.random(d) * 1e-4).astype(np.float32)
    z0 = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    for method in ("qcmd", "qcmd_z", "qrda"):
        ox, oG, oz = x0.copy(), G0.copy(), z0.copy()
        st = GpuState(L, oc, osc, x0, G0, z0)
        with np.errstate(all="ignore"):
            if method == "qrda":
                oracle.step_qrda(oc, osc, d, bucket, ox, oG, oz, 2, 0.1, 1e-4, 1e-8, 2)
                st.qrda(2, 0.1, 1e-4, 1e-8, 2)
            else:
                oracle.step_qcmd(oc, osc, d, bucket, ox, oG, oz if method == "qcmd_z" else None, 0.1, 1e-4, 1e-8, 2)
                st.qcmd(0.1, 1e-4, 1e-8, 2, track_z=method == "qcmd_z")
        x, G, z = st.get()
        for got, want, name in ((x, ox, "x"), (G, oG, "G"), (z, oz, "z")):
            same = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
            assert same.all(), (method, name, int((~same).sum()))


ONE_SCALE_CASES = [(d, M, kind) for d, M in ((70001, 8), (70001, 6), (9000, 1), (4097, 2))
                   for kind in ("close", "wide", "inf")] + \
                  [(4096 * 4100 + 3, 5, "close"), (4096 * 8200 + 17, 4, "close"),
                   (4096 * 16400 + 5, 2, "close")]                             # 2, 4 and 8 tiles per group


@pytest.mark.parametrize("d,M,scales", ONE_SCALE_CASES)
def test_steps_with_one_scale_everywhere_match_oracle(d, M, scales):
    """One scale per message, one for Q(SynQ), few workers: the two sums behind Q(SynQ) come from a
    kernel of their own that builds its tables once per work-group and walks 1, 2, 4 or 8 tiles (by
    the vector's length).  Scales close together take its tables, scales spread over 80 binades
    its worker-ordered sum, an infinite scale poisons the sums; fields of the last code word beyond
    d hold garbage and must not count."""
    rng = np.random.default_rng(d + M)
    g = make_grad("laplace_sparse" if d > 10 ** 6 else "gauss", M, d, seed=7 * d + M)
    if scales != "close":
        g = g * (2.0 ** rng.integers(-40, 40, (M, 1))).astype(np.float32)
    oc, osc, _ = oracle.quantize_pack(g, bucket=0)
    if scales == "inf":
        osc[M // 2, 0] = np.inf
    if d % 16:
        oc[:, -1] |= np.uint32((0xFFFFFFFF << (2 * (d % 16))) & 0xFFFFFFFF)      # garbage past d
    L = qa.Layout.make(d, M, 0)
    x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
    G0 = (rng.random(d) * 1e-4).astype(np.float32)
    z0 = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    for method in ("qcmd", "qcmd_z", "qrda"):
        ox, oG, oz = x0.copy(), G0.copy(), z0.copy()
        st = GpuState(L, oc, osc, x0, G0, z0)
        with np.errstate(all="ignore"):
            if method == "qrda":
                oracle.step_qrda(oc, osc, d, 0, ox, oG, oz, 3, 0.1, 1e-4, 1e-8, 2)
                st.qrda(3, 0.1, 1e-4, 1e-8, 2)
            else:
                oracle.step_qcmd(oc, osc, d, 0, ox, oG, oz if method == "qcmd_z" else None, 0.1, 1e-4, 1e-8, 2)
                st.qcmd(0.1, 1e-4, 1e-8, 2, track_z=method == "qcmd_z")
        x, G, z = st.get()
        for got, want, name in ((x, ox, "x"), (G, oG, "G"), (z, oz, "z")):
            same = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
            assert same.all(), (method, name, int((~same).sum()))


@pytest.mark.parametrize("d,M,bucket,requant", AGGQ_CASES)
def test_aggregate_quantize_matches_oracle_and_the_fused_step(d, M, bucket, requant):
    g = make_grad("gauss", M, d, seed=31 * d + M)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    L = qa.Layout.make(d, M, bucket)
    bq = bucket if requant == 1 else 0
    L1 = qa.Layout.make(d, 1, bq)
    # oracle: the average, then the quantizer on it as a one-worker message
    gbar = oracle.aggregate(oc, osc, d, bucket)
    qc_ref, qs_ref, qt_ref = oracle.quantize_pack(gbar[None, :], bucket=bq)
    codes, scales = dev(oc.view(np.int32)), dev(osc)
    qc = torch.full((1, L1.code_stride), -1, dtype=torch.int32, device=DEV)
    qs = torch.full((1, L1.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    qt = torch.full((1, L1.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    ws = workspace(qa.qa_workspace_bytes(L, qa.QA_OP_STEP))
    qa.qa_aggregate_quantize(L, codes, scales, requant, qc, qs, qt, ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(qc).view(np.uint32)[:, :L1.words], qc_ref)
    assert np.array_equal(host(qs)[:, :L1.n_buckets].view(np.uint32), qs_ref.view(np.uint32))
    assert np.array_equal(host(qt)[:, :L1.n_buckets].view(np.uint32), qt_ref.view(np.uint32))
    # stepping from the message == the fused step with the same second quantization
    rng = np.random.default_rng(d)
    x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
    G0 = (rng.random(d) * 1e-4).astype(np.float32)
    z0 = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    xa, Ga, za = dev(x0), dev(G0), dev(z0)
    xb, Gb, zb = dev(x0), dev(G0), dev(z0)
    qa.qa_step_qrda(L, codes, scales, xa, Ga, za, 3, 0.1, 2e-4, 1e-8, requant, ws)
    qa.qa_step_qrda(L1, qc, qs, xb, Gb, zb, 3, 0.1, 2e-4, 1e-8, qa.QA_REQUANT_NONE, None)
    torch.cuda.synchronize()
    for u, v in ((xa, xb), (Ga, Gb), (za, zb)):
        assert np.array_equal(host(u).view(np.uint32), host(v).view(np.uint32))


def test_aggregate_quantize_checks_its_arguments():
    L = qa.Layout.make(100000, 2, 4096)
    t = torch.zeros(8, dtype=torch.int32, device=DEV)
    f = torch.zeros(8, dtype=torch.float32, device=DEV)
    with pytest.raises(qa.QaError) as e:                 # NONE is not a quantization
        qa.qa_aggregate_quantize(L, t, f, qa.QA_REQUANT_NONE, t, f, None, None)
    assert e.value.code == -1
    with pytest.raises(qa.QaError) as e:                 # one scale for 100000 components needs the workspace
        qa.qa_aggregate_quantize(L, t, f, qa.QA_REQUANT_GLOBAL, t, f, None, None)
    assert e.value.code == -3
    L0 = qa.Layout.make(100000, 2, 0)
    with pytest.raises(qa.QaError) as e:                 # per-bucket needs buckets
        qa.qa_aggregate_quantize(L0, t, f, qa.QA_REQUANT_BUCKET, t, f, None, None)
    assert e.value.code == -1


def one_read_gradient(kind, d, rng):
    g = (rng.standard_normal(d) * 1e-2).astype(np.float32)
    tile = np.arange(d) // 4096
    if kind == "sparse":
        g *= rng.random(d) < 0.05
    elif kind == "trend":                               # magnitudes grow along the vector
        g *= (1.0 + 3.0 * np.arange(d, dtype=np.float32) / d)
    elif kind == "sample misleads":                     # the tiles that are sampled are ten times smaller
        g[np.isin(tile, sampled_tiles(d))] *= np.float32(0.1)
    elif kind == "sample empty":
        g[np.isin(tile, sampled_tiles(d))] = 0
    elif kind == "crowd at the threshold":              # a third of the components within 1e-3 of it
        near = rng.random(d) < 0.33
        mean = np.abs(g[~near]).mean(dtype=np.float64)
        # mean of the mixture m = 0.67 mean + 0.33 * 0.75 m
        delta = 0.75 * 0.67 * mean / (1 - 0.33 * 0.75)
        g[near] = (delta * (1 + 1e-3 * rng.uniform(-1, 1, int(near.sum())))).astype(np.float32)
        g *= np.where(rng.random(d) < 0.5, -1, 1).astype(np.float32)
    elif kind == "rising":                              # all components near the threshold in a few tiles
        g = (np.arange(1, d + 1) * np.where(rng.random(d) < 0.5, -1, 1)).astype(np.float32)
    elif kind == "zero":
        g[:] = 0
    elif kind == "nan":
        g[d // 2] = np.nan
    return g


@pytest.mark.parametrize("kinds,d,bucket", [(("gauss", "sparse"), (1 << 24) + 12345, 0),
                                            (("trend", "sample misleads"), 1 << 24, 0),
                                            (("sample empty", "crowd at the threshold"), (1 << 24) + 1, 0),
                                            (("zero", "nan", "gauss"), (1 << 24) + 4095, 0),
                                            (("rising", "gauss", "rising", "sparse"), (1 << 24) + 70001, 0),
                                            (("gauss",), (1 << 25) + (1 << 23) + 77, 1 << 24)])
def test_quantizer_of_long_buckets_matches_oracle(kinds, d, bucket):
    """Buckets long enough for the form that reads the gradient once (2^24 components, 2^25 in all): where the
    sample brackets the threshold, where it does not, and in an incomplete last bucket; with the smaller
    workspace of the two-read form the message is the same."""
    rng = np.random.default_rng(d % 1000 + len(kinds))
    g = np.stack([one_read_gradient(k, d, rng) for k in kinds])
    M = len(kinds)
    c_ref, s_ref, t_ref = oracle.quantize_pack(g, bucket=bucket)
    c, s, th, L = gpu_quantize_pack(g, bucket)
    nb = L.n_buckets
    same = np.isnan(t_ref) | (ulp_distance(np.nan_to_num(th[:, :nb]), np.nan_to_num(t_ref)) <= 1)
    assert same.all()
    assert np.array_equal(np.isnan(th[:, :nb]), np.isnan(t_ref))
    assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1
    if np.array_equal(np.nan_to_num(th[:, :nb]), np.nan_to_num(t_ref)):
        assert np.array_equal(c[:, :L.words], c_ref)
    else:                                               # a threshold's last bit (2^-29 each): codes for the GPU's own
        assert np.array_equal(c[:, :L.words], oracle.quantize_pack(g, bucket=bucket, thresholds=th[:, :nb])[0])
    gs = (d + 3) // 4 * 4
    gp = np.zeros((M, gs), np.float32); gp[:, :d] = g
    small = workspace(M * ((d + 4095) // 4096) * 12 + M * nb * 4 + 768)
    assert small.numel() < qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
    codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
    scales = torch.zeros((M, L.scale_stride), dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack(L, dev(gp), gs, codes, scales, None, 0, small)
    torch.cuda.synchronize()
    assert np.array_equal(host(codes).view(np.uint32)[:, :L.words], c[:, :L.words])
    assert int(ulp_distance(host(scales)[:, :nb], s[:, :nb]).max()) <= 1


def order_sensitive_gradient(d):
    """One thread's sixteen components of the first tile: a large one whose binary64 sum with each of twelve small
    ones rounds back to it, while the small ones added up first would change it.  With coefficient 1.5 and
    2^k components the threshold is a tie between two binary32 numbers that such a change decides."""
    g = np.zeros(d, np.float32)
    g[0] = (1 + 3 * 2.0 ** -23) * 2.0 ** 30
    for j in (1024, 2048, 3072):
        g[j:j + 4] = 2.0 ** -23
    return g


def test_threshold_does_not_depend_on_the_workspace():
    """The one-read and the two-read form add the magnitudes in the same order."""
    d, M = 1 << 24, 2
    L = qa.Layout.make(d, M, 0, 1.5)
    g = dev(np.stack([order_sensitive_gradient(d)] * M))
    codes = torch.zeros((M, L.code_stride), dtype=torch.int32, device=DEV)
    full = qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
    assert full >= M * (d // 4096) * 20
    got = []
    for size in (full, M * (d // 4096) * 12 + 4 * M + 768):
        sc, th = torch.zeros((2, M, 1), dtype=torch.float32, device=DEV)
        qa.qa_quantize_pack(L, g, d, codes, sc, th, 0, workspace(size))
        torch.cuda.synchronize()
        got.append(host(th))
    assert np.array_equal(*got)
    assert np.array_equal(got[0], oracle.quantize_pack(host(g), bucket=0, thr_coef=1.5)[2])


@pytest.mark.parametrize("bucket", [1 << 25, 1 << 27, 1 << 30])
def test_quantizer_of_a_bucket_far_longer_than_the_vector(bucket):
    """A bucket size beyond the vector's length means one bucket: the same message as with one scale per vector,
    bit for bit, and nothing written outside the workspace."""
    d, M, guard = (1 << 24) + 4099, 2, 1 << 20
    rng = np.random.default_rng(5)
    gs = (d + 3) // 4 * 4
    g = torch.zeros((M, gs), dtype=torch.float32, device=DEV)
    g[:, :d] = dev(rng.standard_normal((M, d), dtype=np.float32))
    messages = []
    for b in (0, bucket):
        L = qa.Layout.make(d, M, b)
        assert L.n_buckets == 1
        size = qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
        ws = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
        codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
        sc, th = torch.zeros((2, M, 1), dtype=torch.float32, device=DEV)
        qa.qa_quantize_pack(L, g, gs, codes, sc, th, 0, ws[:size])
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xA5).all())
        messages.append((codes[:, :L.words], sc, th))
    for a, b in zip(*messages):
        assert torch.equal(a, b)


# ---- exact least-squares threshold by ranking (Section 3.4) ------------------------------------

@pytest.mark.parametrize("d,M,bucket", [(4096, 1, 0), (1000, 2, 0), (3, 1, 0), (4096 * 5, 3, 4096),
                                        (4096 * 7 + 1234, 4, 4096), (4096 * 3 + 1, 2, 4096),
                                        # buckets smaller than the tile: the network stops early
                                        (10000, 2, 64), (10000, 2, 128), (9001, 3, 256), (12289, 2, 512),
                                        (10000, 2, 1024), (4096 * 3 + 77, 3, 2048), (70, 1, 64)])
@pytest.mark.parametrize("kind", ["gauss", "student", "laplace_sparse"])
def test_exact_threshold_quantizer_matches_oracle(d, M, bucket, kind):
    g = make_grad(kind, M, d, seed=d % 977 + M)
    th_ref = np.stack([oracle.exact_thresholds(g[m], bucket) for m in range(M)])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    nb = L.n_buckets
    assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c[:, :L.words], c_ref)
    assert np.array_equal(s[:, :nb].view(np.uint32), s_ref.view(np.uint32))


@pytest.mark.parametrize("bucket", [4096, 256, 64])
def test_exact_threshold_never_splits_equal_magnitudes_and_handles_zeros(bucket):
    rng = np.random.default_rng(5)
    d = 4096 * 3
    g = np.zeros((3, d), np.float32)
    g[0] = rng.integers(-3, 4, d)                       # many ties, many zeros, sums exact
    g[1, ::7] = 2.5                                      # all kept magnitudes equal
    g[2, :4096] = rng.standard_normal(4096)              # all-zero buckets after the first tile
    th_ref = np.stack([oracle.exact_thresholds(g[m], bucket) for m in range(3)])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    assert np.array_equal(th.view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c, c_ref)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32))
    first_empty = 4096 // bucket
    assert th[2, first_empty] == 0 and s[2, first_empty] == 0 and not c[2, 256:].any()


def hard_bucket(kind, n, rng):
    """Magnitudes on which the search for the optimum has little to go by, or much to rank."""
    if kind == "one":                                   # a single non-zero component
        v = np.zeros(n); v[n // 3] = -2.5
    elif kind == "equal":
        v = np.full(n, 0.37)
    elif kind == "two values":                          # equal objectives for one value and for both
        v = np.where(np.arange(n) % 4 == 0, 3.0, 1.0)
    elif kind == "flat":                                # a_k ~ k^-1/2: the objective hardly changes with k
        v = 1.0 / np.sqrt(np.arange(1, n + 1))
    elif kind == "level":                               # S_k = sqrt(k): every cut is as good as any other
        v = np.sqrt(np.arange(1, n + 1)) - np.sqrt(np.arange(n)); v = rng.permutation(v)
    elif kind == "crowded":                             # all magnitudes within one bin's width of each other
        v = 1.0 + rng.random(n) * 1e-5
    elif kind == "two clusters":
        v = np.where(rng.random(n) < 0.5, 1.0 + 0.01 * rng.random(n), 0.2 + 0.01 * rng.random(n))
    elif kind == "outlier":
        v = rng.standard_normal(n) * 1e-3; v[5] = 1e4
    elif kind == "wide":                                # 60 binades
        v = np.exp2(rng.uniform(-40, 20, n))
    elif kind == "tiny":                                # subnormal members
        v = rng.standard_normal(n) * 1e-38
    elif kind == "huge":                                # their binary32 sum overflows
        v = rng.uniform(0.5, 1.0, n) * 3e38
    else:                                               # integers: ties everywhere
        v = rng.integers(-9, 10, n).astype(float)
    return (v * np.where(rng.random(n) < 0.5, -1.0, 1.0)).astype(np.float32)


HARD = ["one", "equal", "two values", "flat", "level", "crowded", "two clusters", "outlier", "wide", "tiny", "huge",
        "integers"]


@pytest.mark.parametrize("bucket,tail", [(4096, 0), (4096, 1), (2048, 4095), (1024, 1023), (1024, 0),
                                         (512, 300)])
def test_exact_threshold_on_hard_buckets(bucket, tail):
    """One kind of bucket after the other in one vector, every kind also in the incomplete last bucket
    (one worker per kind).  Where sums of the kept magnitudes round differently the scale may differ by
    an ulp; the kept set may not."""
    rng = np.random.default_rng(bucket + tail)
    rows = []
    for k in range(len(HARD)):
        kinds = HARD[k:] + HARD[:k]
        parts = [hard_bucket(q, bucket, rng) for q in kinds]
        if tail:
            parts.append(hard_bucket(kinds[-1], tail, rng) if tail > 5 else parts[0][:tail])
        rows.append(np.concatenate(parts))
    g = np.stack(rows)
    th_ref = np.stack([oracle.exact_thresholds(r, bucket) for r in g])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    nb = L.n_buckets
    assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c[:, :L.words], c_ref)
    assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1


def tied_bucket(kind, n, rng):
    """Few different magnitudes, many times each."""
    if kind == "steps":
        v = np.round(rng.standard_normal(n) * 32) / 32
    elif kind == "coarse steps":
        v = np.round(rng.standard_normal(n) * 2)
    elif kind == "one value and zeros":
        v = np.where(rng.random(n) < 0.5, 0.01, 0.0)
    elif kind == "close pair":                          # both kept, nothing below
        v = np.where(rng.random(n) < 0.5, 1.0, 0.9)
    elif kind == "close pair over many small":          # both kept, the threshold lies far below half the mean
        v = np.where(rng.random(n) < 0.9, np.where(rng.random(n) < 0.5, 1.0, 0.9), 0.01 * rng.random(n))
    elif kind == "beside a crowd":                      # one step's members differ in their last bits
        v = np.round(rng.standard_normal(n) * 4) / 4
        v = np.where(np.abs(v) == 0.5, v * (1 + rng.integers(0, 300, n) * 2.0 ** -23), v)
    elif kind == "huge steps":
        v = rng.integers(1, 5, n) * 8e37
    elif kind == "steps of the smallest":
        v = rng.integers(0, 50, n) * 2.0 ** -126
    else:                                               # equal objectives: 1 of the first and all three of the second
        v = np.where(np.arange(n) % 4 == 0, 3.0, 1.0)
    return (v * np.where(rng.random(n) < 0.5, -1.0, 1.0)).astype(np.float32)


TIED = ["steps", "coarse steps", "one value and zeros", "close pair", "close pair over many small", "beside a crowd",
        "huge steps", "steps of the smallest", "equal objectives"]


@pytest.mark.parametrize("bucket", [512, 1024, 2048, 4096])
def test_exact_threshold_on_tied_magnitudes(bucket):
    """More members around the optimum than are ranked one by one, but few values: the cuts between them are
    compared, or the bucket is left to the ranking network where a bin holds several values."""
    rng = np.random.default_rng(bucket)
    for tail in (0, bucket // 2 + 3):
        g = np.stack([np.concatenate([tied_bucket(k, bucket, rng) for k in TIED] + ([tied_bucket(k0, tail, rng)] if tail else []))
                      for k0 in TIED])
        th_ref = np.stack([oracle.exact_thresholds(r, bucket) for r in g])
        c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
        c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
        nb = L.n_buckets
        assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
        assert np.array_equal(c[:, :L.words], c_ref)
        assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1


# buckets longer than one tile, and one threshold for a long vector: device-wide ranking
@pytest.mark.parametrize("d,M,bucket", [(70001, 2, 0), (70001, 2, 8192), (4096 * 5 + 1, 3, 16384),
                                        (4097, 1, 0), (300001, 1, 0), (8192 * 3, 2, 8192),
                                        ((1 << 20) + 17, 1, 65536),
                                        # one bucket that is longer than the vector, buckets ending one
                                        # past a tile, several workers with a padded gradient stride
                                        (5000, 2, 8192), (8193, 3, 8192), (4097, 2, 16384)])
@pytest.mark.parametrize("kind", ["gauss", "student", "laplace_sparse"])
def test_exact_threshold_over_several_tiles_matches_oracle(d, M, bucket, kind):
    """Section 3.4's optimum over a bucket (or a whole gradient) of many tiles.  At these sizes the
    objectives of neighbouring k differ by far more than the rounding of the binary64 sums, so
    the k, and with it threshold, codes and scale, must be the oracle's."""
    g = make_grad(kind, M, d, seed=d % 977 + M)
    th_ref = np.stack([oracle.exact_thresholds(g[m], bucket) for m in range(M)])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    nb = L.n_buckets
    assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c[:, :L.words], c_ref)
    assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1   # binary64 sums over many tiles, rounded once


# chunks of 12 tiles with 10 and with 8 in the last, one chunk per bucket, and more work-groups than compute units
@pytest.mark.parametrize("d,M,bucket", [(4096 * 93 + 17, 32, 0), (5 * (1 << 17) - 100, 16, 1 << 17),
                                        (65540, 256, 0), (65540, 257, 0)])
def test_exact_threshold_at_the_ends_of_its_chunks_matches_oracle(d, M, bucket):
    g = make_grad("gauss", M, d, seed=d % 977 + M)
    th_ref = np.stack([oracle.exact_thresholds(g[m], bucket) for m in range(M)])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    nb = L.n_buckets
    assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c[:, :L.words], c_ref)
    assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1   # binary64 sums over many tiles, rounded once


@pytest.mark.parametrize("bucket", [0, 8192])
def test_exact_threshold_over_several_tiles_with_ties_zeros_and_a_ramp(bucket):
    rng = np.random.default_rng(11)
    d = 8192 * 4 + 300
    g = np.zeros((4, d), np.float32)
    g[0] = rng.integers(-3, 4, d)                       # many ties, many zeros, sums exact
    g[1, ::7] = 2.5                                      # all kept magnitudes equal
    g[2, :5000] = rng.standard_normal(5000)              # all-zero buckets after the first
    g[3] = rng.permutation(np.arange(1, d + 1))          # a ramp: the closed form of the pin
    th_ref = np.stack([oracle.exact_thresholds(g[m], bucket) for m in range(4)])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    assert np.array_equal(th.view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c, c_ref)
    assert np.array_equal(s.view(np.uint32), s_ref.view(np.uint32))
    if bucket:
        assert th[2, 1] == 0 and s[2, 1] == 0 and not c[2, 512:].any()


@pytest.mark.parametrize("bucket,n,tail", [(8192, 8192, 0), (8192, 8192, 4099), (65536, 65536, 3), (0, 9001, 0),
                                           (0, 65537, 0), (131072, 131072, 70001), (0, 300001, 0)])
def test_exact_threshold_over_several_tiles_on_hard_buckets(bucket, n, tail):
    """The same for buckets inside one work-group's reach (up to 65536) and beyond; "level" is what the
    levels of the search cannot narrow down.  Scales within an ulp, the kept sets the oracle's."""
    rng = np.random.default_rng(n + tail)
    kinds = HARD if n < 100000 else ["two values", "level", "wide", "tiny", "integers"]
    rows = []
    for k in range(len(kinds) if bucket == 0 else 2):
        parts = [hard_bucket(q, n, rng) for q in (kinds[k:k + 1] if bucket == 0 else kinds)]
        if tail:
            parts.append(hard_bucket(kinds[k], tail, rng) if tail > 5 else parts[0][:tail])
        rows.append(np.concatenate(parts))
    g = np.stack(rows)
    th_ref = np.stack([oracle.exact_thresholds(r, bucket) for r in g])
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref)
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    nb = L.n_buckets
    assert np.array_equal(th[:, :nb].view(np.uint32), th_ref.view(np.uint32))
    assert np.array_equal(c[:, :L.words], c_ref)
    assert int(ulp_distance(s[:, :nb], s_ref).max()) <= 1


def non_finite_bucket(kind, n, rng):
    v = rng.standard_normal(n).astype(np.float32)
    if kind == "zeros and inf":
        v[:] = 0
    if kind != "nan":
        v[n // 3] = -np.inf
    if kind == "three inf":
        v[[3, n - 1]] = np.inf
    if kind == "largest and inf":
        v[n // 2:] = np.finfo(np.float32).max
    if kind in ("nan", "nan and inf"):
        v[n // 5] = np.nan
    return v


NON_FINITE = ["inf", "three inf", "zeros and inf", "largest and inf", "nan", "nan and inf"]


WIDE_EXACT = [8192, 16384, 65536, 131072]


@pytest.mark.parametrize("bucket", [64, 128, 256, 512, 1024, 2048, 4096] + WIDE_EXACT)
def test_exact_threshold_of_non_finite_buckets(bucket):
    """The objective is infinite as soon as an infinite component is kept, so the smallest k keeps these alone;
    with a NaN there is no optimum and the threshold is 0.  A finite bucket follows each, and the last
    one is incomplete."""
    rng = np.random.default_rng(bucket)
    parts = [p for k in NON_FINITE for p in (non_finite_bucket(k, bucket, rng), rng.standard_normal(bucket).astype(np.float32))]
    for tail in (np.zeros(0, np.float32), non_finite_bucket("three inf", bucket // 2 + 5, rng)):
        g = np.concatenate(parts + [tail])[None]
        th_ref = oracle.exact_thresholds(g[0], bucket)
        for i, k in enumerate(NON_FINITE):
            if "nan" in k:
                th_ref[2 * i] = 0
        c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th_ref[None])
        c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
        nb = L.n_buckets
        assert np.array_equal(th[0, :nb].view(np.uint32), th_ref.view(np.uint32))
        assert np.array_equal(c[:, :L.words], c_ref)
        finite = np.isfinite(s_ref)
        assert np.array_equal(s[:, :nb][~finite], s_ref[~finite], equal_nan=True)
        assert int(ulp_distance(s[:, :nb][finite], s_ref[finite]).max()) <= 1


def test_exact_threshold_of_a_long_vector_is_optimal_to_binary64_resolution():
    """Beyond some 1e7 components the objectives of neighbouring k near the optimum agree to
    binary64 rounding and the association of the sums may decide between them; what must hold
    at any size: the GPU's kept set is {|v| > its threshold}, no candidate the oracle finds is
    better than it by more than that rounding, and codes and scale follow from the threshold."""
    d, M = (1 << 24) + 12345, 1
    g = np.empty((M, d), np.float32)
    g[0] = host(synth.grad_laplace_sparse(d, 0, 1, device=DEV, seed=77, keep=0.5))
    c, s, th, L = gpu_quantize_pack(g, 0, exact=True)
    a = np.abs(g[0].astype(np.float64))
    kept = a > float(th[0, 0])
    k = int(kept.sum())
    assert k > 0 and (th[0, 0] == 0 or (a == float(th[0, 0])).any())      # an actual magnitude
    obj_gpu = a[kept].sum() ** 2 / k
    _, _, obj_ref, k_ref = oracle.exact_threshold(g[0])
    assert obj_gpu >= obj_ref * (1 - 1e-12)
    print(f"\n[exact, d=2^24] kept {k} (oracle {k_ref}), objective ratio - 1 = {obj_gpu / obj_ref - 1:.2e}")
    c_ref, s_ref, _ = oracle.quantize_pack(g, 0, thresholds=th[:, :1])
    assert np.array_equal(c[:, :L.words], c_ref)
    assert int(ulp_distance(s[:, :1], s_ref[:, :1]).max()) <= 1


SAMPLED = ["gauss", "sparse laplace", "layers", "heavy", "ternary", "ramp", "outlier", "inf", "small ones", "zeros", "nan",
           "block"]


def sampled_vector(kind, d, rng):
    v = rng.standard_normal(d).astype(np.float32)
    if kind == "sparse laplace":
        v = (rng.laplace(size=d) * (rng.random(d) < 0.05)).astype(np.float32)
    if kind == "layers":                                 # magnitudes that differ along the vector
        v *= np.repeat(10.0 ** -np.arange(8), -(-d // 8))[:d].astype(np.float32)
    if kind == "heavy":                                  # an optimum of few: no bracket
        v /= rng.standard_normal(d).astype(np.float32)
    if kind == "ternary":                                # an optimum between two values
        v = rng.integers(-1, 2, d).astype(np.float32)
    if kind == "ramp":                                   # the bracket's components lie side by side: the list overflows
        v = np.arange(d, dtype=np.float32)
    if kind == "outlier":                                # beyond the histogram of the one pass
        v[d // 2] = 1e30
    if kind == "inf":
        v[[5, d // 2]] = np.inf
    if kind == "small ones":                             # all but a few below the histogram
        v[rng.random(d) < 0.7] = 1e-20
    if kind == "zeros":
        v[:] = 0
    if kind == "nan":
        v[d - 3] = np.nan
    if kind == "block":                                  # all that is kept in one place
        v *= 1e-6
        v[d // 3: d // 3 + d // 40] *= 1e6
    return v


@pytest.mark.parametrize("d,bucket", [((1 << 21) + 4099, 0), ((1 << 21) + 4099, 1 << 21), (1 << 22, 1 << 21)])
@pytest.mark.parametrize("first", range(0, len(SAMPLED), 4))
def test_exact_threshold_of_sampled_buckets(d, bucket, first):
    """Buckets long enough to be sampled and read once, where the bracket holds and where it does not, next to each
    other.  Thresholds are the oracle's unless two cuts agree to binary64 rounding (2^-52 a term over
    2^22 terms of one sign, of which a few cancel: 1e-12 of the objective)."""
    rng = np.random.default_rng(d + first)
    kinds = SAMPLED[first:first + 4]
    g = np.stack([sampled_vector(k, d, rng) for k in kinds])
    c, s, th, L = gpu_quantize_pack(g, bucket, exact=True)
    b = bucket or d
    for m, kind in enumerate(kinds):
        for k in range(L.n_buckets):
            v = g[m, k * b:(k + 1) * b]
            if np.isnan(v).any():
                assert th[m, k] == 0
                continue
            ref = oracle.exact_thresholds(v)[0]
            if th[m, k] != ref:
                a = np.abs(v.astype(np.float64))
                kept, kept_ref = a > th[m, k], a > ref
                obj, best = a[kept].sum() ** 2 / kept.sum(), a[kept_ref].sum() ** 2 / kept_ref.sum()
                assert (a == th[m, k]).any() and obj >= best * (1 - 1e-12), (kind, k, th[m, k], ref)
    c_ref, s_ref, _ = oracle.quantize_pack(g, bucket, thresholds=th[:, :L.n_buckets])
    assert np.array_equal(c[:, :L.words], c_ref)
    finite = np.isfinite(s_ref)
    assert np.array_equal(s[:, :L.n_buckets][~finite], s_ref[~finite])
    assert int(ulp_distance(s[:, :L.n_buckets][finite], s_ref[finite]).max()) <= 1


def test_exact_threshold_checks_workspace_and_missing_output():
    g = dev(np.ones((1, 8192), np.float32))
    codes = torch.zeros((1, 512), dtype=torch.int32, device=DEV)
    scales = torch.zeros((1, 128), dtype=torch.float32, device=DEV)
    th = torch.zeros((1, 128), dtype=torch.float32, device=DEV)
    for bucket in (8192, 0):                            # buckets beyond one tile need the larger workspace
        L = qa.Layout.make(8192, 1, bucket)
        assert qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE_EXACT) > qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
        ws = workspace(qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE))
        with pytest.raises(qa.QaError) as e:
            qa.qa_quantize_pack(L, g, 8192, codes, scales, th, qa.QA_THRESH_EXACT, ws)
        assert e.value.code == -3
        with pytest.raises(qa.QaError) as e:            # and are refused without it
            qa.qa_quantize_pack_static(L, g, 8192, codes, scales, th, qa.QA_THRESH_EXACT)
        assert e.value.code == -6
    L = qa.Layout.make(8192, 1, 4096)
    assert qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE_EXACT) == qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
    with pytest.raises(qa.QaError) as e:
        qa.qa_quantize_pack(L, g, 8192, codes, scales, None, qa.QA_THRESH_EXACT, None)
    assert e.value.code == -1
    with pytest.raises(qa.QaError) as e:
        qa.qa_quantize_pack(L, g, 8192, codes, scales, th,
                            qa.QA_THRESH_EXACT | qa.QA_THRESH_GIVEN, None)
    assert e.value.code == -1


def crowded(g, tile, groups):
    """Components near the threshold of g in `groups` float4 groups of one wave's quarter of a tile, the rest of it far
    below."""
    delta = np.float32(0.75) * np.abs(g).mean(dtype=np.float64)
    part = g[tile * 4096:(tile + 1) * 4096].reshape(4, 4, 64, 4)          # group index j, wave, lane, component
    part[:, 1] = np.float32(1e-3) * delta
    at = part[:, 1].reshape(-1, 4).copy()
    at[:groups] = np.float32(delta) * np.where(np.arange(4) % 2, np.float32(1.0003), np.float32(-0.9997))
    part[:, 1] = at.reshape(4, 64, 4)


def one_read_without_lists_bytes(L):
    """A workspace for the form with one read that marks what is open in the code words: sums, counts and thresholds of the
    two reads, sums and brackets of the one."""
    def arrays(*sizes):
        return sum((n + 255) // 256 * 256 for n in sizes)
    tiles, nb = (L.d + 4095) // 4096, L.n_buckets
    return arrays(L.M * tiles * 8, L.M * tiles * 4, L.M * nb * 4) + arrays(L.M * tiles * 8, L.M * nb * 8)


@pytest.mark.parametrize("d,bucket", [(1 << 24, 0), ((1 << 24) + 4099, 0), ((1 << 26) + 1, 0),   # one tile of 32 sampled, one of 64
                                      ((1 << 25) + (1 << 24) - 7 * 4096 - 30, 1 << 24)])         # the last bucket shorter
def test_long_quantizer_lists_what_is_open(d, bucket):
    """Lists of 14 float4 groups (the longest), of 15 (the tiles are coded again) and of a whole wave; open components in the
    last, incomplete tile, behind which the row holds other values; a sample that misleads.  Same codes as with two
    reads, same message bit for bit from a call that has no room for lists and marks what is open in its words."""
    rng = np.random.default_rng(11)
    M, gs = 2, (d + 3) // 4 * 4 + 8
    g = (rng.standard_normal((M, d)) * 1e-2).astype(np.float32)
    for tile, groups in ((5, 14), (13, 15), (21, 256), (22, 1), ((d >> 12) - 1, 14)):
        crowded(g[0], tile, groups)
    delta = np.float32(0.75) * np.abs(g[0]).mean(dtype=np.float64)
    g[0, -1] = delta * np.float32(1.0002)
    b = bucket or d
    for lo in range(0, d, b):
        n = min(b, d - lo)
        g[1, lo:lo + n][np.isin(np.arange(n) >> 12, sampled_tiles(b)[sampled_tiles(b) < n >> 12])] *= np.float32(0.5)
    gp = np.full((M, gs), delta, np.float32)              # padding inside the bracket belongs to nobody
    gp[:, :d] = g
    L = qa.Layout.make(d, M, bucket)
    nb, tiles = L.n_buckets, (d + 4095) >> 12
    gd, out = dev(gp), []
    full = qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)
    sizes = {"listed": full, "two reads": M * tiles * 12 + 4 * M * nb + 768, "marked": one_read_without_lists_bytes(L)}
    assert sizes["two reads"] < sizes["marked"] and sizes["marked"] + M * tiles * 128 == full
    for how in ("listed", "two reads", "marked", "static"):
        codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
        sc, th = torch.zeros((2, M, nb), dtype=torch.float32, device=DEV)
        if how == "static":
            qa.qa_quantize_pack_static(L, gd, gs, codes, sc, th, 0)
        else:
            qa.qa_quantize_pack(L, gd, gs, codes, sc, th, 0, workspace(sizes[how]))
        torch.cuda.synchronize()
        out.append((codes[:, :L.words], sc, th))
    for other in out[2:]:
        for one, two in zip(out[0], other):
            assert torch.equal(one, two)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][2], out[1][2])
    assert int(ulp_distance(host(out[0][1]), host(out[1][1])).max()) <= 1
    quantizer_parity(g, bucket, host(out[0][0]).view(np.uint32), host(out[0][1]), host(out[0][2]), (d, bucket))


# buckets of 2 .. 16 tiles are held in registers; 65537 components under one scale are the first that are not
@pytest.mark.parametrize("bucket,d", [(8192, 8193), (8192, 5 * 8192 - 7), (16384, 3 * 16384), (16384, 16384 + 4097), (32768, 2 * 32768 + 4096),
                                      (32768, 20481), (65536, 3 * 65536 - 4095), (65536, 65536 + 1), (65536, 40000),
                                      (0, 4097), (0, 8192), (0, 12291), (0, 32769), (0, 65535), (0, 65536), (0, 65537)])
def test_buckets_held_in_registers_match_oracle_and_the_two_passes(bucket, d):
    """Incomplete last tiles and buckets, buckets longer than the vector; with the thresholds handed in, the passes over
    the gradient give the same message bit for bit (sums added in the same order), also of infinities and NaN."""
    rng = np.random.default_rng(d)
    M = 3
    g = (rng.standard_normal((M, d)) * 10.0 ** rng.integers(-3, 3, (M, d))).astype(np.float32)
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    quantizer_parity(g, bucket, codes, scales, th, (bucket, d))
    assert (codes[:, L.words:] == 0xFFFFFFFF).all() and (scales[:, L.n_buckets:] == -7).all()
    g[0, 7], g[1, d - 1], g[2, :] = np.inf, np.nan, 0
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    other = gpu_quantize_pack(g, bucket, thresholds=th[:, :L.n_buckets])
    assert np.array_equal(codes, other[0])
    assert np.array_equal(scales.view(np.uint32), other[1].view(np.uint32))


# both kernels of the steps: up to 400 tiles of two workers, 256 of more, and 400 to 2048 tiles times workers a work-group
# of 1024 threads takes a tile, beyond them the one with tables
@pytest.mark.parametrize("tiles,M,bucket,requant", [
    (512, 1, 0, 0), (513, 1, 4096, 1), (512, 4, 64, 1), (513, 4, 256, 1), (256, 8, 2048, 1), (257, 8, 1024, 0),
    (128, 16, 65536, 1), (129, 16, 0, 2), (3, 17, 512, 1), (1, 17, 0, 2), (5, 24, 4096, 0), (5, 32, 4096, 1),
    (5, 20, 8192, 0), (2, 64, 128, 1), (400, 2, 256, 1), (401, 2, 4096, 0), (257, 3, 1024, 1), (200, 8, 128, 1), (201, 8, 128, 1),
    (256, 7, 4096, 2), (257, 7, 256, 2), (100, 4, 4096, 2), (101, 4, 1024, 2), (50, 8, 256, 2), (51, 8, 4096, 2),
    (100, 12, 4096, 0), (101, 12, 2048, 1), (40, 16, 256, 1), (41, 16, 256, 1), (100, 8, 1024, 1), (101, 8, 1024, 1),
    (25, 16, 512, 1), (26, 16, 512, 1)])
@pytest.mark.parametrize("method", ["qcmd", "qcmd_z", "qrda"])
def test_steps_on_either_side_of_the_line_of_few_tiles(method, tiles, M, bucket, requant):
    """State with values at the ends of the exponent range next to ordinary ones, an incomplete last tile, garbage in
    the code fields behind it: the oracle's bits from both kernels."""
    d = tiles * 4096 - 4089 + 4 * (M % 5)
    rng = np.random.default_rng(tiles + 31 * M)
    g = make_grad("laplace_sparse", M, d, seed=M)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    if d % 16:
        oc[:, -1] |= np.uint32((0xFFFFFFFF << (2 * (d % 16))) & 0xFFFFFFFF)
    L = qa.Layout.make(d, M, bucket)
    pool = np.array([0.0, -0.0, 1e-45, 1e-40, 1e-35, 1.2e-29, 1.3e-29, 1e-20, 1.0, 1e20, 9e37, 3e38, np.inf, np.nan], np.float32)
    x0 = (rng.standard_normal(d) * 1e-2 * (rng.random(d) < 0.5)).astype(np.float32)
    G0 = (rng.random(d) * 1e-5).astype(np.float32)
    z0 = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    for a, signed in ((x0, True), (G0, False), (z0, True)):
        where = rng.random(d) < 0.01
        v = rng.choice(pool, int(where.sum()))
        a[where] = v * rng.choice([-1, 1], v.size) if signed else np.abs(v)
    ox, oG, oz = x0.copy(), G0.copy(), z0.copy()
    st = GpuState(L, oc, osc, x0, G0, z0)
    with np.errstate(all="ignore"):
        if method == "qrda":
            oracle.step_qrda(oc, osc, d, bucket, ox, oG, oz, 3, 0.1, 2e-4, 1e-8, requant)
            st.qrda(3, 0.1, 2e-4, 1e-8, requant)
        else:
            tz = method == "qcmd_z"
            oracle.step_qcmd(oc, osc, d, bucket, ox, oG, oz if tz else None, 0.1, 2e-4, 1e-8, requant)
            st.qcmd(0.1, 2e-4, 1e-8, requant, track_z=tz)
    for name, a, o in zip("xGz", st.get(), (ox, oG, oz)):
        same = (a.view(np.uint32) == o.view(np.uint32)) | (np.isnan(a) & np.isnan(o))
        assert same.all(), (name, int((~same).sum()), a[~same][:4], o[~same][:4])


@pytest.mark.parametrize("scales", ["close", "wide", "inf"])
@pytest.mark.parametrize("M", [4, 5, 6, 7, 8])
def test_sums_from_counted_combinations_match_oracle(M, scales):
    """5 to 8 workers of at least 1024 tiles, one scale per message: the two sums behind Q(SynQ) from the number of
    coordinates with each combination of codes; an odd number of tiles, a last word that ends inside."""
    test_steps_with_one_scale_everywhere_match_oracle(4096 * 1025 + 4 * M + 1, M, scales)


@pytest.mark.parametrize("tiles,M", [(1024, 7), (16385, 5), (16384, 8)])
def test_counted_combinations_with_crowded_bins_and_reserved_codes(tiles, M):
    """All workers of one mind over most of the vector (one bin takes nearly everything), the pattern 10 among the codes
    (read as 0); step and, from 16384 tiles on, the server's call."""
    d = 4096 * tiles - 5
    rng = np.random.default_rng(tiles + M)
    words = (d + 15) // 16
    oc = np.full((M, words), 0x55555555, np.uint32)
    oc[:, ::3] = rng.integers(0, 1 << 32, (M, (words + 2) // 3), dtype=np.uint32)
    osc = (1e-2 * rng.uniform(0.5, 1.5, (M, 1))).astype(np.float32)
    L = qa.Layout.make(d, M, 0)
    x0 = (rng.standard_normal(d) * 1e-2).astype(np.float32)
    G0 = (rng.random(d) * 1e-4).astype(np.float32)
    ox, oG = x0.copy(), G0.copy()
    oracle.step_qcmd(oc, osc, d, 0, ox, oG, None, 0.1, 1e-4, 1e-8, 2)
    st = GpuState(L, oc, osc, x0, G0, np.zeros(1, np.float32))
    st.qcmd(0.1, 1e-4, 1e-8, 2, track_z=False)
    x, G, _ = st.get()
    assert np.array_equal(x, ox) and np.array_equal(G, oG)
    if tiles >= 16384:
        avg = oracle.aggregate(oc, osc, d, 0)
        c_ref, s_ref, t_ref = oracle.quantize_pack(avg[None], bucket=0)
        q = torch.zeros((1, words), dtype=torch.int32, device=DEV)
        qs, qt = torch.zeros((2, 1, 1), dtype=torch.float32, device=DEV)
        qa.qa_aggregate_quantize(L, dev(oc.view(np.int32)), dev(osc), 2, q, qs, qt,
                                 workspace(qa.qa_workspace_bytes(L, qa.QA_OP_STEP)))
        torch.cuda.synchronize()
        assert np.array_equal(host(qs), s_ref) and np.array_equal(host(qt), t_ref)
        assert np.array_equal(host(q).view(np.uint32), c_ref)


# rows of code words that begin on 64 bytes are stored through the cache, others (up to 7 * 2^24 components) not
@pytest.mark.parametrize("d", [4096 * 65 - 9, 4096 * 33 + 4])
@pytest.mark.parametrize("bucket", [0, 256, 4096])
@pytest.mark.parametrize("first,between", [(0, 0), (0, 3), (16, 0), (1, 0), (5, 8)])
def test_code_words_of_rows_that_begin_anywhere(d, bucket, first, between):
    """The message does not depend on where the rows begin, and the words around a row stay as they were; two reads with
    one scale."""
    M = 5
    g = make_grad("gauss", M, d, seed=d % 97)
    L = qa.Layout.make(d, M, bucket, code_stride=(d + 15) // 256 * 16 + 16 + between)
    gs = (d + 3) // 4 * 4
    gp = np.zeros((M, gs), np.float32)
    gp[:, :d] = g
    buf = torch.full((first + M * L.code_stride + 64,), -1, dtype=torch.int32, device=DEV)
    scales, th = torch.zeros((2, M, L.scale_stride), dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack(L, dev(gp), gs, buf[first:], scales, th, 0, workspace(qa.qa_workspace_bytes(L, qa.QA_OP_QUANTIZE)))
    torch.cuda.synchronize()
    buf = host(buf).view(np.uint32)
    rows = buf[first:first + M * L.code_stride].reshape(M, -1)
    quantizer_parity(g, bucket, rows, host(scales), host(th), (bucket, d, first, between))
    assert (buf[:first] == 0xFFFFFFFF).all() and (buf[first + M * L.code_stride:] == 0xFFFFFFFF).all()
    assert (rows[:, L.words:] == 0xFFFFFFFF).all()


# the average and its second quantization: few tiles and few workers, one more of either
@pytest.mark.parametrize("tiles,M,bucket", [(128, 7, 4096), (129, 7, 4096), (128, 4, 0), (129, 4, 256), (200, 3, 4096), (201, 3, 0),
                                            (256, 2, 256), (257, 2, 128), (5, 8, 1024), (1, 2, 64), (1, 1, 0)])
def test_server_on_either_side_of_the_line_of_few_tiles(tiles, M, bucket):
    """qa_aggregate_unpack, and qa_aggregate_quantize with a scale per bucket and with one: the oracle's bits (one scale for
    several tiles: its sums in another order)."""
    d = tiles * 4096 - 4089 + 4 * M
    rng = np.random.default_rng(tiles + M)
    g = make_grad("student", M, d, seed=M)
    oc, osc, _ = oracle.quantize_pack(g, bucket=bucket)
    avg = oracle.aggregate(oc, osc, d, bucket)
    L = qa.Layout.make(d, M, bucket)
    codes, scales = dev(oc.view(np.int32)), dev(osc)
    out = torch.full(((d + 3) // 4 * 4 + 4,), 7.0, dtype=torch.float32, device=DEV)
    qa.qa_aggregate_unpack(L, codes, scales, out)
    torch.cuda.synchronize()
    assert np.array_equal(host(out)[:d].view(np.uint32), avg.view(np.uint32)) and (host(out)[d:] == 7).all()
    for requant, b in ((qa.QA_REQUANT_BUCKET, bucket), (qa.QA_REQUANT_GLOBAL, 0)):
        if requant == qa.QA_REQUANT_BUCKET and bucket == 0:
            continue
        q = torch.full((1, L.words + 4), -1, dtype=torch.int32, device=DEV)
        qs, qt = torch.full((2, 1, oracle.n_buckets(d, b) + 4), -7.0, dtype=torch.float32, device=DEV)
        qa.qa_aggregate_quantize(L, codes, scales, requant, q, qs, qt, workspace(qa.qa_workspace_bytes(L, qa.QA_OP_STEP)))
        torch.cuda.synchronize()
        quantizer_parity(avg[None], b, host(q).view(np.uint32), host(qs), host(qt), (tiles, M, b))
        assert (host(q)[:, L.words:] == -1).all() and (host(qs)[:, oracle.n_buckets(d, b):] == -7).all()


# 12 tiles are held from 24 work-groups on, 13 from 36, 16 from 72
@pytest.mark.parametrize("bucket,d,M", [(0, 45057, 23), (0, 45057, 24), (0, 49157, 35), (0, 49157, 36), (65536, 3 * 65536 - 5, 23),
                                        (65536, 3 * 65536 - 5, 24), (65536, 61441, 59), (65536, 61441, 72)])
def test_long_buckets_on_either_side_of_the_line_of_held_ones(bucket, d, M):
    """The oracle's message, and with the thresholds handed in (two passes on either side) the same one bit for bit."""
    rng = np.random.default_rng(M)
    g = (rng.standard_normal((M, d)) * 10.0 ** rng.integers(-3, 3, (M, 1))).astype(np.float32)
    codes, scales, th, L = gpu_quantize_pack(g, bucket)
    quantizer_parity(g, bucket, codes, scales, th, (bucket, d, M))
    other = gpu_quantize_pack(g, bucket, thresholds=th[:, :L.n_buckets])
    assert np.array_equal(codes, other[0])
    assert np.array_equal(scales.view(np.uint32), other[1].view(np.uint32))


# 6 tiles are always held, 7 from 42 work-groups on, 16 from 96; otherwise the maxima come from a pass of their own
@pytest.mark.parametrize("bucket,d,M", [(0, 24577, 41), (0, 24577, 42), (0, 24576, 1), (32768, 5 * 32768 - 9, 9), (32768, 5 * 32768 - 9, 10),
                                        (65536, 3 * 65536 - 5, 31), (65536, 3 * 65536 - 5, 32), (65536, 61441, 2)])
def test_stochastic_quantizer_on_either_side_of_the_line_of_held_buckets(bucket, d, M):
    """The oracle's message: scales from whole buckets and the incomplete last one, a bucket of zeros, NaN."""
    rng = np.random.default_rng(d + M)
    g = rng.standard_normal((M, d), dtype=np.float32)
    g[0, :bucket or d], g[M - 1, d - 1], g[M - 1, 7] = 0, np.nan, -9
    oc, osc = oracle.quantize_pack_stochastic(g, bucket=bucket, seed=3, step=7)
    L, gs = qa.Layout.make(d, M, bucket), (d + 3) // 4 * 4
    gp = np.full((M, gs), 99, np.float32)                 # padding belongs to nobody
    gp[:, :d] = g
    codes = torch.full((M, L.code_stride), -1, dtype=torch.int32, device=DEV)
    scales = torch.full((M, L.scale_stride), -7.0, dtype=torch.float32, device=DEV)
    qa.qa_quantize_pack_stochastic(L, dev(gp), gs, codes, scales, 3, 7)
    torch.cuda.synchronize()
    assert np.array_equal(host(scales), osc)
    assert np.array_equal(host(codes).view(np.uint32), oc)
