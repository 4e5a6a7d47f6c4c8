"""Frame-resident launches of more frames than the device holds at once.

Several frames then share a CU, workgroups draw their frames from the launch's
queue, and the kernel instances without address tables in LDS run, none of
which a launch of a few frames reaches.  Each batch must equal, bit for bit,
the streaming kernels' decoding of the same frames: K copies of the code along
the diagonal are too large for the frame-resident kernel, and every copy's
rows, columns and message orders are the code's own.  No tolerance: both
evaluate each message with the same operations in the same order.
"""
import numpy as np
import pytest

from test_gpu_decode_routes import LDS_WORDS, _stack
from workloads import codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1812_06545_amd as lib
    return lib


def _compare(L, name, code, td, frames, iters, es, **kw):
    import torch
    K = LDS_WORDS // code.edges + 1
    small, big = L.Code.from_workload(code), L.Code.from_workload(_stack(code, K))
    assert L.ldpc_batch_fits_fused(small, td)[0] and not L.ldpc_batch_fits_fused(big, td)[0]
    # With early stop every copy holds the same frame, so the stacked frame
    # stops where the small one does; the frames' noise differs, so some stop
    # at once and some never.
    rng = np.random.default_rng(46)
    shape = (frames, code.n) if es else (-(-frames // K), K * code.n)
    x = 3.0 + np.linspace(0.2, 3.0, shape[0])[:, None] * rng.standard_normal(shape)
    t = torch.from_numpy(x.astype(np.float32)).cuda().to(td)
    print(f"[gpu] shared {name} {td} {kw} frames={frames} es={es}", flush=True)
    one = t if es else t.reshape(-1, code.n)
    job = L.Job(small, one.contiguous(), iters, early_stop=es, **kw)
    L.decode_batch([job])
    stacked = t.repeat(1, K) if es else t
    bits, its, post = L.decode(big, stacked.contiguous(), iters, early_stop=es, **kw)
    if es:
        stops = its.tolist()
        assert torch.equal(job.iters, its) and len(set(stops)) > 2
        bits, post = bits[:, :code.n], post[:, :code.n]
    assert torch.equal(bits.reshape(job.bits.shape), job.bits) and torch.equal(post.reshape(job.posterior.shape), job.posterior)


# six groups of rows on eight wavefronts, two frames to a CU: the wavefronts
# swap places from layer to layer; five groups, three frames, and one frame of
# ten groups: they keep them
LAYERED = {"two_frames": (12, 81), "three_frames": (8, 66), "one_frame": (6, 160)}


@pytest.mark.parametrize("es", [False, True])
@pytest.mark.parametrize("name", list(LAYERED))
def test_layered(L, name, es):
    import torch
    mb, Z = LAYERED[name]
    _compare(L, name, codes.qc_code(mb, 24, Z, 47), torch.float32, 700, 4, es, layered=True)


# rows of each degree bucket of the frame-resident kernel
DEGREES = {
    "d8": lambda: codes.random_rows(170, 400, 3, 8, 711),
    "d16": lambda: codes.qc_row_degrees([16, 14, 12, 10, 9, 9], 16, 27, 701),
    "d24": lambda: codes.qc_row_degrees([24, 22, 20, 18, 17], 24, 27, 702),
    "d32": lambda: codes.random_rows(40, 400, 25, 32, 705, dense_col=True),
}
RULES = {
    "flooding": {},
    "layered": dict(layered=True),
    "minsum": dict(rule="minsum", ms_scale=0.8125, ms_offset=0.25),
    "layered_minsum": dict(layered=True, rule="minsum"),
}


@pytest.mark.parametrize("rule", list(RULES))
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("name", list(DEGREES))
def test_degree_buckets(L, name, dtype, rule):
    """More frames of a short code than the device holds at once in any instance
    (24 wavefronts a CU in workgroups of two)."""
    import torch
    td = torch.float32 if dtype == "f32" else torch.float64
    for es in (False, True):
        _compare(L, name, DEGREES[name](), td, 3300, 4, es, **RULES[rule])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_jobs_of_every_kind(L, dtype):
    """One launch of jobs of every schedule, rule and bucket, drawn from one queue,
    against each job's own launch."""
    import torch
    td = torch.float32 if dtype == "f32" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(52)

    def jobs_of():
        return [L.Job(h, x, 5, early_stop=es, **kw) for h, x, es, kw in specs]
    specs = []
    for i, make in enumerate(DEGREES.values()):
        code = make()
        h = L.Code.from_workload(code)
        for k, kw in enumerate(RULES.values()):
            x = 2.5 + 1.7 * torch.randn((150 + 37 * k + i, code.n), generator=gen, device="cuda", dtype=torch.float64)
            specs.append((h, x.to(td), (i + k) % 2 == 0, kw))
    print(f"[gpu] shared: jobs of every kind {dtype}", flush=True)
    together, alone = jobs_of(), jobs_of()
    L.decode_batch(together)
    for job in alone:
        L.decode_batch([job])
    for a, b in zip(together, alone):
        assert torch.equal(a.bits, b.bits) and torch.equal(a.iters, b.iters) and torch.equal(a.posterior, b.posterior)
