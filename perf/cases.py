"""Decoding calls whose speed is watched, over the range that users of the library meet.

A case is a dict of plain values.  `entry` names the public call ("decode", "batch", "plan" or
"server"), `code` the family of parity-check matrices, `frames` how many frames one call decodes; the
rest are the call's own options.  Codes are the families of the repository's workloads and tests:

  qc       quasi-cyclic, mb x 24 base matrix lifted by Z (lengths 24 Z; mb = 12, 8, 6, 4 for rates
           1/2, 2/3, 3/4, 5/6)
  mix      several such codes in one call
  gallager (3,6)-regular
  rows     irregular, row degrees dmin .. dmax, no structure
  stair    rate-1/2 irregular with a dual-diagonal parity part, for the long lengths

Inputs are random codewords sent as BPSK over an AWGN channel.  A code's matrix and encoder are made
once per process; frames, noise, handles, plans, workspaces and servers are made by every `prepare`.
"""
import functools
import math

import numpy as np
import torch

import paper_1812_06545_amd as ldpc
from workloads import codes as matrices
from workloads import gf2

R_MAX = 20.0
MIX = tuple((mb, Z) for Z in (27, 54, 81) for mb in (12, 8, 6, 4))


def _case(name, entry, code, frames, iters, stop, ebn0, *, mb=12, Z=81, n=0, dmin=0, dmax=0, kinds=12, layered=False,
          rule="spa", scale=1.0, offset=0.0, dtype="f32", code_seed=201):
    c = dict(entry=entry, code=code, frames=frames, iters=iters, stop=stop, ebn0=ebn0, layered=layered, rule=rule,
             scale=scale, offset=offset, dtype=dtype, code_seed=code_seed)
    if code == "qc":
        c.update(mb=mb, Z=Z)
    elif code == "mix":
        c.update(kinds=kinds)
    else:
        c.update(n=n)
        if code == "rows":
            c.update(dmin=dmin, dmax=dmax)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short control frame that a caller waits for: launches and latency
        _case("one_frame", "decode", "qc", 1, 10, True, 2.0, mb=12, Z=27),
        # a handful of frames of a link's current code, layered because it converges in fewer passes
        _case("few_layered", "decode", "qc", 24, 10, True, 2.5, mb=8, Z=54, layered=True),
        # the benchmark's batch: throughput decoding of one code, a fixed number of iterations
        _case("stream_4096", "decode", "qc", 4096, 10, False, 2.0),
        # a base station's mixed traffic: twelve codes in one call
        _case("mix_16384", "batch", "mix", 16384, 10, True, 2.0, kinds=12),
        # throughput decoding on the layered schedule with early stop
        _case("layered_4096", "batch", "qc", 4096, 20, True, 3.5, layered=True),
        # normalised min-sum, the usual hardware rule, on an odd batch
        _case("minsum_1999", "batch", "qc", 1999, 10, False, 2.0, rule="minsum", scale=0.75),
        # reference-precision decoding of a regular code (simulation work)
        _case("gallager_f64", "decode", "gallager", 1000, 20, True, 2.0, n=504, dtype="f64", code_seed=101),
        # broadcast-length frames, the longest decodes
        _case("long_256", "decode", "stair", 256, 50, True, 1.0, n=64800, code_seed=501),
        # a few long frames that a caller waits for
        _case("long_few", "decode", "stair", 5, 50, True, 1.2, n=16200, code_seed=502),
        # an unstructured irregular code at an odd length and batch
        _case("rows_333", "decode", "rows", 333, 15, False, 3.0, n=1999, dmin=2, dmax=29, code_seed=705),
        # a receiver loop that replays one captured launch sequence over its four current codes
        _case("plan_64", "plan", "mix", 64, 10, True, 2.0, kinds=4),
        # a burst of requests of up to 64 frames from host buffers
        _case("serve_burst", "server", "mix", 512, 10, True, 2.0, kinds=12),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(("qc", "qc", "qc", "mix", "gallager", "rows", "stair"))
    seed, f64 = rng.randrange(1, 1 << 20), rng.random() < 0.2
    stop = rng.random() < 0.6
    kw = dict(layered=rng.random() < 0.3, dtype="f64" if f64 else "f32", code_seed=seed)
    if rng.random() < 0.3:
        kw.update(rule="minsum", scale=rng.choice((1.0, 0.75, 0.8125)), offset=rng.choice((0.0, 0.0, 0.25)))
    ebn0, entry = round(rng.uniform(1.0, 4.0), 2), rng.choice(("decode", "decode", "batch", "plan"))
    most, iters = (512 if f64 else 4096), rng.randint(3, 12)
    if family == "qc":
        Z = rng.randint(24, 160)
        return _case(None, entry, "qc", _log_int(rng, 1, most * 81 // max(81, Z)), iters, stop, ebn0,
                     mb=rng.choice((12, 8, 6, 4)), Z=Z, **kw)
    if family == "mix":
        kinds = rng.randint(2, 12)
        return _case(None, rng.choice(("batch", "plan")), "mix", _log_int(rng, kinds, 4 * most), iters, stop, ebn0,
                     kinds=kinds, **kw)
    if family == "gallager":
        return _case(None, entry, "gallager", _log_int(rng, 1, most // 4 if kw["layered"] else most), iters, stop, ebn0,
                     n=6 * rng.randint(30, 340), **kw)
    if family == "rows":
        n = rng.randint(200, 2600)
        dmax = rng.choice((8, 16, 24, 32, 40))
        kw["layered"] = False
        return _case(None, entry, "rows", _log_int(rng, 1, most // 2), iters, stop, ebn0, n=n, dmin=max(2, dmax // 2 - 4),
                     dmax=dmax, **kw)
    n = 10 * _log_int(rng, 200, 6480)
    kw.update(layered=False, dtype="f32")
    return _case(None, "decode", "stair", _log_int(rng, 1, min(2048, 256 * 64800 // n)), rng.randint(8, 50), stop,
                 round(rng.uniform(0.8, 2.0), 2), n=n, **kw)


# ------------------------------------------------------------------ matrices --

class _Matrix:
    """A parity-check matrix and its encoder, on the host."""

    def __init__(self, code, encoder):
        self.code, self.encoder = code, encoder
        self.rate = 1.0 - code.m / code.n


@functools.lru_cache(maxsize=64)
def _matrix(family, a, b, c, d, seed):
    if family == "stair":
        return _Matrix(matrices.staircase_irregular(a, seed), None)
    if family == "qc":
        code = matrices.qc_code(a, 24, b, seed)
    elif family == "gallager":
        code = matrices.gallager_regular(a, 3, 6, seed)
    else:
        code = matrices.random_rows(int(a * 0.4), a, b, c, seed)
    return _Matrix(code, gf2.SystematicEncoder(code.to_dense()))


def _parts(case):
    """[(matrix, frames)] of the jobs of one call."""
    f = case["code"]
    if f == "mix":
        kinds, total = case["kinds"], case["frames"]
        order = np.random.RandomState(case["code_seed"]).permutation(len(MIX))[:kinds]
        weight = 1 + np.arange(kinds)
        frames = np.maximum(1, total * weight // weight.sum())
        frames[-1] = max(1, total - int(frames[:-1].sum()))
        return [(_matrix("qc", MIX[k][0], MIX[k][1], 0, 0, 301 + int(k)), int(x)) for k, x in zip(order, frames)]
    if f == "qc":
        return [(_matrix("qc", case["mb"], case["Z"], 0, 0, case["code_seed"]), case["frames"])]
    return [(_matrix(f, case["n"], case.get("dmin", 0), case.get("dmax", 0), 0, case["code_seed"]), case["frames"])]


# -------------------------------------------------------------------- inputs --

def _codewords(mx, frames, gen):
    code, enc = mx.code, mx.encoder
    if enc is None:  # dual-diagonal parity part: row i gives p_i = s_i xor p_(i-1), s_i from its five info columns
        u = torch.randint(0, 2, (frames, code.m), generator=gen, device="cuda", dtype=torch.uint8)
        info = torch.from_numpy(code.col_idx[code.col_idx < code.m].reshape(code.m, 5).astype(np.int64)).cuda()
        s = torch.zeros((frames, code.m), dtype=torch.int32, device="cuda")
        for k in range(5):
            s += u[:, info[:, k]]
        p = torch.cumsum(s, 1) & 1
        return torch.cat([u, p.to(torch.uint8)], 1)
    u = torch.randint(0, 2, (frames, enc.k), generator=gen, device="cuda", dtype=torch.uint8)
    cw = torch.zeros((frames, code.n), dtype=torch.uint8, device="cuda")
    cw[:, torch.from_numpy(enc.info).cuda()] = u
    if enc.pivots.size:
        parity = u.float() @ torch.from_numpy(np.ascontiguousarray(enc.A.T)).cuda()  # whole numbers below 2^24: exact
        cw[:, torch.from_numpy(enc.pivots).cuda()] = (parity.round().to(torch.int32) & 1).to(torch.uint8)
    return cw


def _inputs(case, seed):
    """[(matrix, LLRs)] of the jobs, on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 13)
    out = []
    for mx, frames in _parts(case):
        cw = _codewords(mx, frames, gen)
        sigma2 = 1.0 / (2.0 * mx.rate * 10.0 ** (case["ebn0"] / 10.0))
        noise = torch.randn(cw.shape, generator=gen, device="cuda", dtype=torch.float64)
        llr = (2.0 / sigma2) * (1.0 - 2.0 * cw.double() + math.sqrt(sigma2) * noise)
        out.append((mx, llr if case["dtype"] == "f64" else llr.float()))
    return out


class _Server:
    """A server, its codes and one burst of requests in host memory."""

    def __init__(self, case, inputs):
        self.codes = [ldpc.Code.from_workload(mx.code) for mx, _ in inputs]
        self.handle = ldpc.ldpc_server_create(self.codes, 64 << 20, max_inflight=3, max_group_frames=1024)
        self.requests = []
        self.outputs = []
        for k, (mx, llr) in enumerate(inputs):
            host = llr.cpu().numpy()
            frames, n = host.shape
            bits, its = np.zeros((frames, n), np.uint8), np.zeros(frames, np.int32)
            post = np.zeros((frames, n), np.float32)
            self.outputs.append((bits, its, post))
            at, size = 0, 1
            while at < frames:  # requests of 1 .. 64 frames
                to = min(frames, at + size)
                self.requests.append((k, to - at, host[at:to], bits[at:to], its[at:to], post[at:to]))
                at, size = to, 1 + (size * 5 + 11) % 64
        self.iters, self.flags = case["iters"], ldpc.LDPC_EARLY_STOP if case["stop"] else 0

    def run(self):
        tickets = []
        for k, frames, llr, bits, its, post in self.requests:
            status, ticket = ldpc.ldpc_server_submit(self.handle, k, frames, self.iters, self.flags, llr, bits, its, post)
            if status != ldpc.LDPC_OK:
                raise ldpc.LdpcError(status, "ldpc_server_submit")
            tickets.append(ticket)
        for ticket in tickets:
            status = ldpc.ldpc_server_wait(self.handle, ticket)
            if status != ldpc.LDPC_OK:
                raise ldpc.LdpcError(status, "ldpc_server_wait")
        return self.outputs

    def __del__(self):
        if getattr(self, "handle", None):
            ldpc.ldpc_server_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    inputs = _inputs(case, seed)
    state = {"case": case, "entry": case["entry"]}
    if case["entry"] == "server":
        state["server"] = _Server(case, inputs)
        return state
    codes = [ldpc.Code.from_workload(mx.code) for mx, _ in inputs]
    options = dict(early_stop=case["stop"], layered=case["layered"], rule=case["rule"], ms_scale=case["scale"],
                   ms_offset=case["offset"])
    if case["entry"] == "decode":
        (_, llr), code = inputs[0], codes[0]
        need = ldpc.ldpc_workspace_bytes(code, llr.dtype, llr.shape[0], case["iters"])
        state.update(code=code, llr=llr, options=options,
                     workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
        return state
    jobs = [ldpc.Job(code, llr, case["iters"], **options) for code, (_, llr) in zip(codes, inputs)]
    state["jobs"] = jobs
    if case["entry"] == "plan":
        state["plan"] = ldpc.Plan(jobs)
    else:
        need = ldpc.ldpc_batch_workspace_bytes([j.c_struct() for j in jobs], jobs[0].llr.dtype)
        state["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    entry = state["entry"]
    if entry == "decode":
        bits, iters, post = ldpc.decode(state["code"], state["llr"], state["case"]["iters"], workspace=state["workspace"],
                                        **state["options"])
        return [(bits, iters, post)]
    if entry == "server":
        return state["server"].run()
    if entry == "plan":
        state["plan"].launch()
    else:
        ldpc.decode_batch(state["jobs"], workspace=state["workspace"])
    return [(j.bits, j.iters, j.posterior) for j in state["jobs"]]


def work(case):
    """LLRs in, bits, counts and posteriors out; per edge and iteration the operations of the check rule (sum-product:
    a subtraction, tanh, the exclusive products, atanh and the column's addition; min-sum: subtraction, two minima, a
    selection, signs and the addition).  Early stop runs about two thirds of the iterations at these noise levels."""
    size = 8 if case["dtype"] == "f64" else 4
    nbytes = flops = 0.0
    iters = case["iters"] * (2.0 / 3.0 if case["stop"] else 1.0)
    per_edge = 10.0 if case["rule"] == "minsum" else 36.0
    for mx, frames in _parts(case):
        nbytes += frames * (mx.code.n * (2.0 * size + 1.0) + 4.0)
        flops += frames * mx.code.edges * iters * per_edge
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------------- 64-bit reference --

def _phi(x):
    e = torch.exp(-x)
    return torch.log1p(2.0 * e / -torch.expm1(-x))


def _messages(q, real, case):
    """Check-to-variable messages of rows q [frames, rows, d] (64 bits); `real` [rows, d] marks the edges."""
    inf = float("inf")
    neg = (q < 0) & real
    odd = (neg.sum(-1, keepdim=True) - neg.long()) & 1
    if case["rule"] == "minsum":
        mag = torch.where(real, q.abs(), inf)
        two, at = torch.topk(mag, min(2, mag.shape[-1]), dim=-1, largest=False)
        second = two[..., 1:2] if two.shape[-1] > 1 else torch.full_like(two[..., :1], inf)
        here = torch.arange(q.shape[-1], device=q.device)
        low = torch.where(here == at[..., :1], second, two[..., :1])
        scale, offset = float(np.float32(case["scale"])), float(np.float32(case["offset"]))
        r = torch.clamp(scale * low - offset, 0.0, R_MAX)
    else:
        f = torch.where(real, _phi(q.abs()), 0.0)
        before = torch.zeros_like(f)
        before[..., 1:] = torch.cumsum(f, -1)[..., :-1]
        after = torch.zeros_like(f)
        after[..., :-1] = torch.cumsum(f.flip(-1), -1).flip(-1)[..., 1:]
        r = torch.clamp(_phi(before + after), max=R_MAX)
    return torch.where(odd == 1, -r, r)


def _layers(code):
    """Runs of consecutive rows that share no column."""
    mark, start, out = np.full(code.n, -1), 0, []
    for i in range(code.m):
        cols = code.col_idx[code.row_ptr[i]:code.row_ptr[i + 1]]
        if (mark[cols] >= start).any():
            out.append((start, i))
            start = i
        mark[cols] = i
    out.append((start, code.m))
    return out


def _reference(code, llr, case):
    dev, F, n, m = llr.device, llr.shape[0], code.n, code.m
    deg = np.diff(code.row_ptr)
    width = int(deg.max())
    cols = np.full((m, width), n, np.int64)
    real = np.arange(width)[None, :] < deg[:, None]
    cols[real] = code.col_idx
    cols, real = torch.from_numpy(cols).to(dev), torch.from_numpy(real).to(dev)
    order = torch.argsort(cols.reshape(-1), stable=True)[: int(code.row_ptr[-1])]
    column = cols.reshape(-1)[order]
    channel = torch.cat([llr.double(), torch.zeros((F, 1), dtype=torch.float64, device=dev)], 1)
    L = channel.clone()
    r = torch.zeros((F, m, width), dtype=torch.float64, device=dev)
    iters = torch.full((F,), case["iters"], dtype=torch.int32, device=dev)
    live = torch.arange(F, device=dev)
    layers = _layers(code) if case["layered"] else None

    def codeword(L):
        bad = torch.zeros(L.shape[0], dtype=torch.bool, device=dev)
        bits = L < 0
        bits[:, n] = False
        odd = torch.zeros((L.shape[0], m), dtype=torch.bool, device=dev)
        for k in range(width):
            odd ^= bits[:, cols[:, k]]
        bad |= odd.any(1)
        return ~bad

    run_L, run_r, run_ch = L, r, channel
    for t in range(case["iters"] + 1):
        if case["stop"] and t < case["iters"]:
            stops = codeword(run_L)
            if bool(stops.any()):
                L[live[stops]] = run_L[stops]
                iters[live[stops]] = t
                keep = ~stops
                live, run_L, run_r, run_ch = live[keep], run_L[keep], run_r[keep], run_ch[keep]
                if live.numel() == 0:
                    break
        if t == case["iters"]:
            break
        if layers is None:
            run_r = torch.where(real, _messages(run_L[:, cols] - run_r, real, case), 0.0)
            run_L = run_ch.index_add(1, column, run_r.reshape(run_r.shape[0], -1)[:, order])
        else:
            run_L, run_r = run_L.clone(), run_r.clone()
            for a, b in layers:
                q = run_L[:, cols[a:b]] - run_r[:, a:b]
                new = torch.where(real[a:b], _messages(q, real[a:b], case), 0.0)
                run_r[:, a:b] = new
                run_L[:, cols[a:b][real[a:b]]] = (q + new)[:, real[a:b]]
    if live.numel():
        L[live] = run_L
    L = L[:, :n]
    return (L < 0).to(torch.uint8), iters, L


def exact(case, seed):
    if case["iters"] * sum(f * mx.code.edges for mx, f in _parts(case)) > 3.5e9:
        return None
    out = []
    for mx, llr in _inputs(case, seed):
        step = max(1, int(4e7) // max(1, int(mx.code.m * np.diff(mx.code.row_ptr).max())))  # frames at a time
        parts = [_reference(mx.code, llr[at:at + step], case) for at in range(0, llr.shape[0], step)]
        out.append(tuple(torch.cat(x) for x in zip(*parts)))
    return out
