"""Parity of the tensor-list entry points (one flat vector holding many tensors, each quantized
on its own) with the CPU oracle, through the C ABI.  Codes, scales, thresholds and zero sets must
be bit-exact; state is asserted within 1e-5 (and is bit-exact in practice)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2208_05631_amd as qa
    from gpu_util import DEV, dev, host, sampled_pieces, workspace

RTOL = 1e-5


def layout_of(lengths, gaps=(0, 1, 3)):
    begin, pos = [], 0
    for i, n in enumerate(lengths):
        begin.append(pos)
        pos = (pos + n + 15) // 16 * 16 + 16 * gaps[i % len(gaps)]
    return np.array(begin, np.int64), np.array(lengths, np.int64), pos + 7


CASES = {
    "mixed": [150, 6, 2400, 16, 0, 48000, 120, 1, 10, 4097, 33],
    "many_small_in_one_tile": [16] * 40 + [5] * 30 + [100] * 20,
    "conv_net_like": [1 * 5 * 5 * 6, 6, 6 * 5 * 5 * 16, 16, 400 * 120, 120, 120 * 84, 84, 84 * 10, 10],
    "one_large": [3 * 4096 + 77],
    "tile_aligned": [4096, 8192, 4096],
    "all_empty": [0, 0, 0],
}


def close(a, b, what):
    if np.array_equal(a, b):
        return
    err = np.max(np.abs(a.astype(np.float64) - b) / np.maximum(np.abs(b), 1e-30))
    assert err <= RTOL, f"{what}: max rel err {err}"


class Flat:
    def __init__(self, lengths, M, seed):
        self.begin, self.length, self.d = layout_of(lengths)
        self.M, self.nseg = M, len(lengths)
        rng = np.random.default_rng(seed)
        self.rng = rng
        self.tensor_scale = 10.0 ** rng.integers(-4, 2, self.nseg)
        self.covered = np.zeros(self.d, bool)
        for b, n in zip(self.begin, self.length):
            self.covered[b:b + n] = True
        self.L = qa.Layout.make(self.d, M, 0, 0.75, None, self.nseg)
        self.table = torch.zeros(qa.qa_segment_plan_bytes(self.d, self.nseg), dtype=torch.uint8, device=DEV)
        self.plan = qa.qa_segment_plan_init(self.d, self.begin, self.length, self.table)
        self.gs = (self.d + 3) // 4 * 4

    def grads(self):
        g = self.rng.standard_normal((self.M, self.d)) * 0.5            # junk between tensors too
        for k, (b, n) in enumerate(zip(self.begin, self.length)):
            g[:, b:b + n] *= self.tensor_scale[k]
            g[:, b:b + n] *= self.rng.random((self.M, n)) < 0.7          # some exact zeros
        return g.astype(np.float32)

    def gpu_quantize(self, g):
        gp = np.zeros((self.M, self.gs), np.float32)
        gp[:, :self.d] = g
        codes = torch.full((self.M, self.L.code_stride), 0x5A5A5A5A, dtype=torch.int32, device=DEV)
        scales = torch.full((self.M, self.nseg), -7.0, dtype=torch.float32, device=DEV)
        th = torch.full((self.M, self.nseg), -7.0, dtype=torch.float32, device=DEV)
        ws = workspace(qa.qa_segment_workspace_bytes(self.plan, self.M, qa.QA_OP_QUANTIZE))
        qa.qa_quantize_pack_segments(self.L, self.plan, dev(gp), self.gs, codes, scales, th, ws)
        torch.cuda.synchronize()
        return codes, scales, th


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("M", [1, 3, 8])
def test_quantize_pack_segments_matches_oracle(case, M):
    f = Flat(CASES[case], M, seed=len(case) + M)
    g = f.grads()
    c_ref, s_ref, th_ref = oracle.quantize_pack_segments(g, f.begin, f.length)
    codes, scales, th = f.gpu_quantize(g)
    c = host(codes).view(np.uint32)
    touched = np.zeros(f.L.words, bool)
    for b, n in zip(f.begin, f.length):
        touched[b // 16:(b + n + 15) // 16] = True
    assert np.array_equal(c[:, touched], c_ref[:, touched])
    assert (c[:, ~touched] == 0x5A5A5A5A).all()                         # left alone
    assert np.array_equal(host(scales).view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(host(th).view(np.uint32), th_ref.view(np.uint32))


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("M,requant", [(1, False), (4, False), (4, True), (8, True), (6, False)])
def test_steps_over_segments_match_oracle(case, M, requant):
    f = Flat(CASES[case], M, seed=7 * len(case) + M)
    rng = f.rng
    for method in ("qcmd_z", "qcmd", "qrda"):
        x = (rng.standard_normal(f.d) * 0.05).astype(np.float32)
        G = (rng.random(f.d) * 1e-3).astype(np.float32)
        z = (rng.standard_normal(f.d) * 0.01).astype(np.float32)
        xr, Gr, zr = x.copy(), G.copy(), z.copy()
        xd, Gd, zd = dev(x), dev(G), dev(z)
        ws = workspace(qa.qa_segment_workspace_bytes(f.plan, M, qa.QA_OP_STEP))
        rq = qa.QA_REQUANT_BUCKET if requant else qa.QA_REQUANT_NONE
        for t in range(1, 4):
            g = f.grads()
            c_ref, s_ref, _ = oracle.quantize_pack_segments(g, f.begin, f.length)
            codes, scales, _ = f.gpu_quantize(g)
            if method == "qrda":
                oracle.step_segments(oracle.QRDA, c_ref, s_ref, f.d, f.begin, f.length, xr, Gr, zr, t,
                                     0.1, 1e-3, 1e-8, requant)
                qa.qa_step_qrda_segments(f.L, f.plan, codes, scales, xd, Gd, zd, t, 0.1, 1e-3, 1e-8, rq, ws)
            else:
                zz = zr if method == "qcmd_z" else None
                oracle.step_segments(oracle.QCMD, c_ref, s_ref, f.d, f.begin, f.length, xr, Gr, zz, t,
                                     0.1, 1e-3, 1e-8, requant)
                qa.qa_step_qcmd_segments(f.L, f.plan, codes, scales, xd, Gd,
                                         zd if method == "qcmd_z" else None, 0.1, 1e-3, 1e-8, rq, ws)
            torch.cuda.synchronize()
            xg, Gg, zg = host(xd), host(Gd), host(zd)
            what = f"{case} {method} M={M} requant={requant} t={t}"
            assert np.array_equal(xg == 0, xr == 0), what                # zero set: exact
            close(xg, xr, what + " x"); close(Gg, Gr, what + " G"); close(zg, zr, what + " z")
            assert np.array_equal(xg[~f.covered], x[~f.covered])         # between tensors: untouched
            assert np.array_equal(Gg[~f.covered], G[~f.covered])
            assert np.array_equal(zg[~f.covered], z[~f.covered])


def test_segment_calls_reject_what_they_cannot_do():
    f = Flat(CASES["mixed"], 2, seed=1)
    g = f.grads()
    codes, scales, _ = f.gpu_quantize(g)
    x = torch.zeros(f.gs, dtype=torch.float32, device=DEV)
    G = torch.zeros(f.gs, dtype=torch.float32, device=DEV)
    ws = workspace(qa.qa_segment_workspace_bytes(f.plan, 2, qa.QA_OP_STEP))
    with pytest.raises(qa.QaError) as e:
        qa.qa_step_qcmd_segments(f.L, f.plan, codes, scales, x, G, None, 0.1, 0.0, 1e-8,
                                 qa.QA_REQUANT_GLOBAL, ws)
    assert e.value.code == -5
    with pytest.raises(qa.QaError) as e:                                # second quantization needs ws
        qa.qa_step_qcmd_segments(f.L, f.plan, codes, scales, x, G, None, 0.1, 0.0, 1e-8,
                                 qa.QA_REQUANT_BUCKET, None)
    assert e.value.code == -3
    Lb = qa.Layout.make(f.d, 2, 4096, 0.75, None, max(f.nseg, (f.d + 4095) // 4096))
    with pytest.raises(qa.QaError) as e:                                # buckets and tensors do not mix
        qa.qa_step_qcmd_segments(Lb, f.plan, codes, scales, x, G, None, 0.1, 0.0, 1e-8, 0, None)
    assert e.value.code == -1
    Ls = qa.Layout.make(f.d, 2, 0, 0.75, None, f.nseg - 1)
    with pytest.raises(qa.QaError) as e:                                # a scale per tensor is needed
        qa.qa_step_qcmd_segments(Ls, f.plan, codes, scales, x, G, None, 0.1, 0.0, 1e-8, 0, None)
    assert e.value.code == -1
    Ld = qa.Layout.make(f.d + 16, 2, 0, 0.75, None, f.nseg)
    with pytest.raises(qa.QaError) as e:                                # plan of another vector
        qa.qa_step_qcmd_segments(Ld, f.plan, codes, scales, x, G, None, 0.1, 0.0, 1e-8, 0, None)
    assert e.value.code == -1


def check_codes(f, g, c, th, c_ref, th_ref):
    """Every tensor's codes: the oracle's where the threshold is the oracle's, else the oracle's for the GPU's own
    threshold.  No field holds the pattern 10, which marks a component still to be decided."""
    for s, (b, n) in enumerate(zip(f.begin, f.length)):
        words = slice(int(b) // 16, (int(b) + int(n) + 15) // 16)
        assert not np.any((c[:, words] >> 1) & ~c[:, words] & 0x55555555), s
        for m in range(f.M):
            expected = c_ref[m, words]
            if th[m, s] != th_ref[m, s]:
                own = np.array([[th[m, s]]], np.float32)
                expected = oracle.quantize_pack(g[m:m + 1, b:b + n], bucket=0, thresholds=own)[0][0]
            assert np.array_equal(c[m, words], expected), (m, s)


@pytest.mark.parametrize("M", [8, 9])
def test_long_tensors_read_once_match_oracle(M):
    """Lists large enough for the form that reads long tensors' gradients once (2^27 components in all):
    tensors just below and above the length that is sampled, one whose sampled pieces mislead, sparse
    and constant ones, small ones between them; steps with the second quantization on top."""
    lengths = [30, 1024 * 4096 - 4096, 17, 1024 * 4096 + 5, 2_000_000, 1100 * 4096, 3, 1500 * 4096 + 1, 100]
    f = Flat.__new__(Flat)
    f.begin, f.length, f.d = layout_of(lengths)
    f.M, f.nseg = M, len(lengths)
    f.L = qa.Layout.make(f.d, M, 0, 0.75, None, f.nseg)
    f.table = torch.zeros(qa.qa_segment_plan_bytes(f.d, f.nseg), dtype=torch.uint8, device=DEV)
    f.plan = qa.qa_segment_plan_init(f.d, f.begin, f.length, f.table)
    f.gs = (f.d + 3) // 4 * 4
    assert f.plan.n_pieces * M >= 32768
    rng = np.random.default_rng(M)
    g = rng.standard_normal((M, f.d), dtype=np.float32)
    t5, pieces = f.begin[5] // 4096, (f.begin[5] + f.length[5] - 1) // 4096 - f.begin[5] // 4096 + 1
    for p in sampled_pieces(pieces):                     # tensor 5: the sampled pieces are ten times larger
        if 0 < p < pieces - 1:
            g[:M // 2, (t5 + p) * 4096:(t5 + p + 1) * 4096] *= 10
    s7 = slice(int(f.begin[7]), int(f.begin[7]) + int(f.length[7]))
    g[0, s7] *= rng.random(f.length[7]) < 0.05
    g[1, s7] = 0.25
    g[2, s7] = 0
    g[3, s7] = np.arange(f.length[7], dtype=np.float32) * np.float32(1e-3)     # open components in a few pieces
    c_ref, s_ref, th_ref = oracle.quantize_pack_segments(g, f.begin, f.length)
    codes, scales, th = f.gpu_quantize(g)
    c = host(codes).view(np.uint32)
    touched = np.zeros(f.L.words, bool)
    for b, n in zip(f.begin, f.length):
        touched[b // 16:(b + n + 15) // 16] = True
    # sums in another order: thresholds and scales within an ulp, codes those of the thresholds
    assert np.allclose(host(th), th_ref, rtol=1.3e-7, atol=0)
    assert np.allclose(host(scales), s_ref, rtol=1.3e-7, atol=0)
    check_codes(f, g, c, host(th), c_ref, th_ref)
    assert (c[:, ~touched] == 0x5A5A5A5A).all()
    x, G, z = (np.zeros(f.d, np.float32) for _ in range(3))
    xd, Gd, zd = dev(x), dev(G), dev(z)
    ws = workspace(qa.qa_segment_workspace_bytes(f.plan, M, qa.QA_OP_STEP))
    oracle.step_segments(oracle.QRDA, c_ref, s_ref, f.d, f.begin, f.length, x, G, z, 1, 0.1, 1e-3, 1e-8, True)
    qa.qa_step_qrda_segments(f.L, f.plan, dev(c_ref.view(np.int32)), dev(s_ref), xd, Gd, zd, 1, 0.1, 1e-3, 1e-8,
                             qa.QA_REQUANT_BUCKET, ws)
    torch.cuda.synchronize()
    for a, r in ((xd, x), (Gd, G), (zd, z)):
        close(host(a)[f_covered(f)], r[f_covered(f)], "state")


@pytest.mark.parametrize("kind", ["gauss", "misled", "sparse"])
def test_tensors_on_either_side_of_the_sampled_lengths_match_oracle(kind):
    """Lists read once: tensors around 128, 256 and 512 pieces (sampled every 4th, 8th, 16th piece, shorter ones not at
    all), whole tiles and not; with the sampled pieces larger than the others the threshold leaves its bracket."""
    lengths = [5, 127 * 4096, 128 * 4096, 130 * 4096 - 9, 255 * 4096 + 7, 256 * 4096, 511 * 4096 - 80, 512 * 4096 + 1, 150 * 4096]
    f = Flat.__new__(Flat)
    f.begin, f.length, f.d = layout_of(lengths)
    f.M, f.nseg = 16, len(lengths)
    f.L = qa.Layout.make(f.d, f.M, 0, 0.75, None, f.nseg)
    f.table = torch.zeros(qa.qa_segment_plan_bytes(f.d, f.nseg), dtype=torch.uint8, device=DEV)
    f.plan = qa.qa_segment_plan_init(f.d, f.begin, f.length, f.table)
    f.gs = (f.d + 3) // 4 * 4
    assert f.plan.n_pieces * f.M >= 32768 and f.plan.n_pieces >= 128 * f.nseg
    rng = np.random.default_rng(len(kind))
    g = rng.standard_normal((f.M, f.d), dtype=np.float32)
    if kind == "sparse":
        g *= rng.random((f.M, f.d), dtype=np.float32) < 0.05
    if kind == "misled":
        for b, n in zip(f.begin, f.length):
            t0, pieces = b // 4096, (b + n - 1) // 4096 - b // 4096 + 1
            for p in sampled_pieces(pieces):
                if 0 < p < pieces - 1:
                    g[::2, (t0 + p) * 4096:(t0 + p + 1) * 4096] *= 1.5
    c_ref, s_ref, th_ref = oracle.quantize_pack_segments(g, f.begin, f.length)
    codes, scales, th = f.gpu_quantize(g)
    # sums in another order: thresholds and scales within an ulp, codes those of the thresholds
    assert np.allclose(host(th), th_ref, rtol=1.3e-7, atol=0)
    assert np.allclose(host(scales), s_ref, rtol=1.3e-7, atol=0)
    check_codes(f, g, host(codes).view(np.uint32), host(th), c_ref, th_ref)


def test_threshold_of_a_long_tensor_does_not_depend_on_the_workspace():
    """The one-read and the two-read form add the magnitudes in the same order: a gradient whose threshold, a tie
    between two binary32 numbers, is decided by the order of a few additions."""
    n, M = 1 << 24, 8
    L = qa.Layout.make(n, M, 0, 1.5, None, 1)
    table = torch.zeros(qa.qa_segment_plan_bytes(n, 1), dtype=torch.uint8, device=DEV)
    plan = qa.qa_segment_plan_init(n, np.zeros(1, np.int64), np.array([n], np.int64), table)
    v = np.zeros(n, np.float32)
    v[0] = (1 + 3 * 2.0 ** -23) * 2.0 ** 30
    for j in (1024, 2048, 3072):
        v[j:j + 4] = 2.0 ** -23
    g = dev(v).repeat(M, 1)
    codes = torch.zeros((M, L.code_stride), dtype=torch.int32, device=DEV)
    full = qa.qa_segment_workspace_bytes(plan, M, qa.QA_OP_QUANTIZE)
    assert full >= M * plan.n_pieces * 20
    got = []
    for size in (full, M * plan.n_pieces * 12 + 4 * M + 768):
        sc, th = torch.zeros((2, M, 1), dtype=torch.float32, device=DEV)
        qa.qa_quantize_pack_segments(L, plan, g, n, codes, sc, th, workspace(size))
        torch.cuda.synchronize()
        got.append(host(th))
    assert np.array_equal(*got)
    assert np.array_equal(got[0][0], oracle.quantize_pack(v[None], bucket=0, thr_coef=1.5)[2][0])


def test_long_tensors_ending_at_every_place_of_a_work_group():
    """Long tensors (read once, settled eight pieces at a time) with one-piece tensors behind them, which the
    same work-group codes right after it has summed what the long one keeps: the boundary at each of the
    eight places.  Several calls give the same bits (sums in a fixed order)."""
    lengths = []
    for k in range(8):
        lengths += [1024 * 4096, 100 + k]
    # every tensor starts on a tile of its own, so that its pieces are whole tiles
    begin = np.cumsum([0] + [-(-n // 4096) * 4096 for n in lengths])
    f = Flat.__new__(Flat)
    f.begin, f.length, f.d = begin[:-1].astype(np.int64), np.array(lengths, np.int64), int(begin[-1])
    f.M, f.nseg = 4, len(lengths)
    f.L = qa.Layout.make(f.d, f.M, 0, 0.75, None, f.nseg)
    f.table = torch.zeros(qa.qa_segment_plan_bytes(f.d, f.nseg), dtype=torch.uint8, device=DEV)
    f.plan = qa.qa_segment_plan_init(f.d, f.begin, f.length, f.table)
    f.gs = f.d
    assert f.plan.n_pieces * f.M >= 32768
    ends = {int((b + n - 1) // 4096) % 8 for b, n in zip(f.begin, f.length) if n > 4096}
    assert ends == set(range(8))
    g = np.random.default_rng(3).standard_normal((f.M, f.d), dtype=np.float32)
    c_ref, s_ref, th_ref = oracle.quantize_pack_segments(g, f.begin, f.length)
    first = None
    for _ in range(4):
        codes, scales, th = f.gpu_quantize(g)
        if first is None:
            first = codes, scales, th
            # sums in another order: an ulp
            assert np.allclose(host(th), th_ref, rtol=1.3e-7, atol=0)
            assert np.allclose(host(scales), s_ref, rtol=1.3e-7, atol=0)
            check_codes(f, g, host(codes).view(np.uint32), host(th), c_ref, th_ref)
        for a, b in zip(first, (codes, scales, th)):
            assert torch.equal(a, b)


def f_covered(f):
    covered = np.zeros(f.d, bool)
    for b, n in zip(f.begin, f.length):
        covered[b:b + n] = True
    return covered
