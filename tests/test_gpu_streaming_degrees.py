"""GPU parity of the streaming kernels, for every degree bucket.

ldpc_decode runs a code that fits the frame-resident kernel there, so the codes
of degree_cases reach the streaming kernels' bodies for rows of up to 32 edges
only stacked: K copies along the diagonal, too large for that kernel.  Every copy
holds the same frame and must give the same outputs; the first copy's are
compared with the oracle, with the bars and horizons of parity_util.

200 frames are three 64-frame chunks and a ragged tail of 8, more than the
few-frames path takes.
"""
import numpy as np
import pytest

import oracle
from degree_cases import FRAMES, FUSED_FITS, workload
from parity_util import HORIZON_F32, compare, compare_horizon
from test_gpu_decode_routes import LDS_WORDS, _stack
from workloads import codes, configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1812_06545_amd as lib
    return lib


def _decode_stacked(L, code, llr, K, T, es, **kw):
    """(bits, iterations, posteriors) of the first copy; the others must equal it."""
    import torch
    h = L.Code.from_workload(_stack(code, K))
    x = torch.from_numpy(np.ascontiguousarray(llr)).cuda()
    assert not L.ldpc_batch_fits_fused(h, x.dtype)[0]
    bits, iters, post = L.decode(h, x.repeat(1, K).contiguous(), T, early_stop=es, **kw)
    bits, post = bits.view(-1, K, code.n), post.view(-1, K, code.n)
    assert (bits == bits[:, :1]).all() and (post == post[:, :1]).all()
    return bits[:, 0].cpu().numpy(), iters.cpu().numpy(), post[:, 0].cpu().numpy()


def _against_oracle(where, code, llr, T, es, got, layered=False):
    schedule = "layered" if layered else "flooding"
    ref = oracle.decode(code, llr, T, es, nthreads=8, schedule=schedule)
    horizon = HORIZON_F32[schedule]
    if llr.dtype == np.float32 and T > horizon:
        compare_horizon(ref, *got, llr.dtype, where, code, T, horizon)
    else:
        compare(ref, *got, llr.dtype, where)


@pytest.mark.parametrize("layered", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FUSED_FITS))
def test_sum_product(L, name, dtype, layered):
    code, llr = workload(name, dtype)
    K = LDS_WORDS // code.edges + 1
    for T, es in ((5, False), (20, True)):
        where = f"streaming {name} {dtype} layered={layered} T={T}"
        print(f"[gpu] {where}", flush=True)
        got = _decode_stacked(L, code, llr, K, T, es, layered=layered)
        _against_oracle(where, code, llr, T, es, got, layered)
        if es:
            assert 0 < (got[1] < T).sum() < FRAMES or name.startswith("spc"), "inputs should mix stops and non-stops"


@pytest.mark.parametrize("layered", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(FUSED_FITS))
def test_minsum(L, name, dtype, layered):
    """FP64 bit for bit, FP32 within the iterations at which its bar holds."""
    code, llr = workload(name, dtype)
    K = LDS_WORDS // code.edges + 1
    T, es = (20, True) if dtype == "f64" else (1 if layered else 4, False)
    print(f"[gpu] streaming min-sum {name} {dtype} layered={layered} T={T}", flush=True)
    bits, iters, post = _decode_stacked(L, code, llr, K, T, es, layered=layered, rule="minsum", ms_scale=0.75)
    ref = oracle.decode(code, llr, T, es, nthreads=8, schedule="layered" if layered else "flooding", rule="minsum",
                        ms_scale=0.75)
    if dtype == "f64":
        assert np.array_equal(iters, ref["iters"]) and np.array_equal(bits, ref["bits"])
        assert np.array_equal(post, ref["posterior"])
    else:
        compare(ref, bits, iters, post, llr.dtype, f"streaming min-sum {name}")


# the row groups from which a block of the check kernel takes two
TWO_GROUPS = {"d8": 8000, "qc_d16": 20000}


@pytest.mark.parametrize("es", [False, True])
@pytest.mark.parametrize("name", list(TWO_GROUPS))
def test_two_row_groups_a_block(L, name, es):
    """Launches of which a block of the check kernel takes two row groups: an odd
    number of groups and a last one of fewer than four rows."""
    if name == "d8":
        code = codes.random_rows(135, 400, 3, 8, 707)
        llr = (2.5 + 1.6 * np.random.default_rng(708).standard_normal((FRAMES, code.n))).astype(np.float32)
    else:
        code, llr = workload(name, "f32")
    chunks = -(-FRAMES // 64)
    K = next(k for k in range(1, 400) if code.m * k % 4 and -(-code.m * k // 4) % 2
             and -(-code.m * k // 4) * chunks >= TWO_GROUPS[name])
    T = 20 if es else 4
    print(f"[gpu] two row groups a block: {name} K={K} es={es}", flush=True)
    got = _decode_stacked(L, code, llr, K, T, es)
    _against_oracle(f"two row groups {name}", code, llr, T, es, got)


@pytest.mark.parametrize("mode", ["flooding", "layered", "min-sum"])
def test_general_instance(L, mode):
    """A job whose code fits the frame-resident kernel only with its messages in CSR
    order makes the whole batch run the general instance: the other jobs' outputs
    stay those of their own instance, and its own are those of ldpc_decode."""
    import torch
    kw = {"flooding": {}, "layered": dict(layered=True), "min-sum": dict(rule="minsum", ms_scale=0.75)}[mode]
    mix = configs.qc_mix(total=720)[::3]
    hs = [L.Code.from_workload(m.code) for m in mix]
    code = codes.random_rows(10900, 6000, 3, 3, 37)  # rows of 3 pad to 4: 171 KB against 154
    h = L.Code.from_workload(code)
    assert L.ldpc_batch_fits_fused(h, torch.float32)[0]
    rng = np.random.default_rng(709)
    x = torch.from_numpy(rng.normal(2.0, 1.8, size=(5, code.n)).astype(np.float32)).cuda()
    for es in (True, False):
        def jobs_of():
            return [L.Job(k, torch.from_numpy(np.ascontiguousarray(m.llr)).cuda(), 6, early_stop=es, **kw)
                    for k, m in zip(hs, mix)]
        print(f"[gpu] general instance {mode} es={es}", flush=True)
        alone, together, extra = jobs_of(), jobs_of(), L.Job(h, x, 3, early_stop=es, **kw)
        L.decode_batch(alone)
        L.decode_batch(together + [extra])
        for a, b in zip(alone, together):
            assert torch.equal(a.bits, b.bits) and torch.equal(a.iters, b.iters) and torch.equal(a.posterior, b.posterior)
        own = L.decode(h, x, 3, early_stop=es, **kw)
        assert torch.equal(own[0], extra.bits) and torch.equal(own[1], extra.iters) and torch.equal(own[2], extra.posterior)
