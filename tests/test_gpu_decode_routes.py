"""ldpc_decode's two routes, frame-resident and streaming, give the same bits.

A code small enough for the frame-resident kernel is stacked K times along
the diagonal, K large enough that the stacked code's messages exceed a
workgroup's LDS: the small code's decode takes the frame-resident kernel, the
stacked one's the streaming kernels, and each copy's rows, columns and
message orders are the small code's.  So every copy's outputs must equal the
small decode's bit for bit (no tolerance: both routes evaluate each message
with the same operations in the same order).  With early stop every copy
holds the same frame, so the stacked frame stops where the small one does.
Frame counts straddle the 64-frame chunks of the streaming layout.
"""
import numpy as np
import pytest

from workloads import codes

pytestmark = pytest.mark.gpu

LDS_WORDS = 160 * 1024 // 4


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1812_06545_amd as lib
    return lib


def _stack(code, K):
    rows = [int(e) * code.edges for e in range(K)]
    row_ptr = np.concatenate([code.row_ptr[:-1].astype(np.int64) + r for r in rows] + [[K * code.edges]])
    col_idx = np.concatenate([code.col_idx.astype(np.int64) + k * code.n for k in range(K)])
    return codes.Code(K * code.m, K * code.n, row_ptr.astype(np.int32), col_idx.astype(np.int32))


# `half`: the message is 8 bytes, so half as many fit.
CODES = {
    "qc_z27": lambda half: codes.qc_code(12, 24, 27, 31),
    "qc_z81_r56": lambda half: codes.qc_code(4, 24, 81, 32),
    "gallager": lambda half: codes.gallager_regular(240, 3, 6, 33),
    "rows_2_29": lambda half: codes.random_rows(120, 311, 2, 29, 34),
    "rows_31_32": lambda half: codes.random_rows(33, 130, 31, 32, 38),
    "rows_dense_col": lambda half: codes.random_rows(70, 190, 1, 16, 35, dense_col=True),
    # rows of degree 3 pad to 4: the messages fit a workgroup's LDS in CSR order only
    "csr_order": lambda half: codes.random_rows(5400, 3000, 3, 3, 37) if half else codes.random_rows(10900, 6000, 3, 3, 37),
}


@pytest.mark.parametrize("rule", ["spa", "minsum"])
@pytest.mark.parametrize("layered", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", list(CODES))
def test_routes_agree(L, name, dtype, layered, rule):
    import torch
    code = CODES[name](dtype == "f64")
    K = LDS_WORDS // code.edges + 1
    small, big = L.Code.from_workload(code), L.Code.from_workload(_stack(code, K))
    td = torch.float32 if dtype == "f32" else torch.float64
    assert L.ldpc_batch_fits_fused(small, td)[0] and not L.ldpc_batch_fits_fused(big, td)[0]
    kw = dict(layered=layered, rule=rule, ms_scale=0.8125, ms_offset=0.25)
    rng = np.random.default_rng(36)
    for frames, es, iters in ((3, False, 3), (70, True, 7)):
        print(f"[gpu] routes {name} {dtype} layered={layered} {rule} frames={frames} es={es}", flush=True)
        x = rng.normal(2.0, 2.2, size=(frames * (1 if es else K), code.n)).astype(np.float32)
        t = torch.from_numpy(x).cuda().to(td)
        bits, its, post = L.decode(small, t, iters, early_stop=es, **kw)
        stacked = t.repeat(1, K) if es else t.reshape(frames, K * code.n)
        b2, i2, p2 = L.decode(big, stacked.contiguous(), iters, early_stop=es, **kw)
        if es:
            assert torch.equal(its, i2)
            bits, post = bits.repeat(1, K), post.repeat(1, K)
        assert torch.equal(b2.reshape(bits.shape), bits) and torch.equal(p2.reshape(post.shape), post)


FEW = {
    "stair": lambda: codes.staircase_irregular(12960, 41),
    "rows_2_16": lambda: codes.random_rows(6001, 12007, 2, 16, 42),
    "rows_dense_col": lambda: codes.random_rows(2503, 5003, 17, 31, 43, dense_col=True),
}


@pytest.mark.parametrize("rule", ["spa", "minsum"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", list(FEW))
def test_few_frames_match_many(L, name, dtype, rule):
    """Up to 32 frames of a code that streams take one launch per iteration, more
    frames the check and variable kernels: a frame decodes to the same bits in
    both, whatever the number of frames beside it, with and without early stop,
    from none to several iterations."""
    import torch
    code = FEW[name]()
    h = L.Code.from_workload(code)
    td = torch.float32 if dtype == "f32" else torch.float64
    assert not L.ldpc_batch_fits_fused(h, td)[0]
    rng = np.random.default_rng(44)
    x = rng.normal(3.0, 1.8, size=(70, code.n)).astype(np.float32)
    x[::5] = np.abs(x[::5])  # codewords from the start: these stop at once
    t = torch.from_numpy(x).cuda().to(td)
    for iters, es in ((0, True), (1, True), (4, False), (9, True)):
        kw = dict(early_stop=es, rule=rule, ms_scale=0.75)
        want = L.decode(h, t, iters, **kw)
        for frames in (1, 5, 8, 11, 32):
            print(f"[gpu] few {name} {dtype} {rule} T={iters} es={es} frames={frames}", flush=True)
            got = L.decode(h, t[:frames].contiguous(), iters, **kw)
            for a, b in zip(got, want):
                assert torch.equal(a, b[:frames])
        if es and iters == 9:
            assert len(set(want[1].tolist())) > 1


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_buffers(L, shift):
    """Frames are moved by fours where n and the pointers allow it: buffers that
    start `shift` elements off a 16-byte boundary (and, for the bits, `shift`
    bytes off a word) give the aligned buffers' outputs, and nothing before or
    behind them is written."""
    import torch
    code = codes.qc_code(12, 24, 27, 31)
    h = L.Code.from_workload(code)
    rng = np.random.default_rng(45)
    frames, n = 9, code.n
    x = torch.from_numpy(rng.normal(2.0, 2.0, size=(frames, n)).astype(np.float32)).cuda()
    for layered in (False, True):
        want = L.Job(h, x, 5, early_stop=True, layered=layered)
        L.decode_batch([want])
        print(f"[gpu] unaligned shift={shift} layered={layered}", flush=True)

        def off(dtype, fill):
            whole = torch.full((frames * n + 8,), fill, dtype=dtype, device="cuda")
            return whole, whole[shift:shift + frames * n].view(frames, n)
        for moved in ("llr", "bits", "posterior", "all"):
            job = L.Job(h, x, 5, early_stop=True, layered=layered)
            edges = []
            if moved in ("llr", "all"):
                _, job.llr = off(torch.float32, 0.0)
                job.llr.copy_(x)
            if moved in ("bits", "all"):
                whole, job.bits = off(torch.uint8, 7)
                edges.append(whole)
            if moved in ("posterior", "all"):
                whole, job.posterior = off(torch.float32, 7.0)
                edges.append(whole)
            L.decode_batch([job])
            torch.cuda.synchronize()
            assert torch.equal(job.bits, want.bits) and torch.equal(job.iters, want.iters)
            assert torch.equal(job.posterior, want.posterior)
            for whole in edges:
                assert (whole[:shift] == 7).all() and (whole[shift + frames * n:] == 7).all()
