"""The work this library is used for, as cases that can be timed.

Each case goes through the public binding (``paper_2609_09800_amd.hbf``) the
way a caller does.  Input streams have the shapes of
``paper_2609_09800_amd.workloads`` (page runs, MoE decode weight streaming,
the mixed stream with a shared KV prefix) but are drawn on the GPU, so that
large ones are made quickly; every draw comes from the seed alone.

Kinds:
  time      reset + hbf_time_requests (the main path), on every media variant
  layers    reset + hbf_time_layers (closed-loop decode)
  refresh   reset + hbf_refresh_submit + hbf_time_requests
  capacity  reset + hbf_cache_access (frame cache with prefetcher)
  gemv      hbf_gemv_instrumented, without delays or with some experts faulted
  classify  hbf_classify_map alone
"""
import math

import numpy as np
import torch

from paper_2609_09800_amd import hbf
from paper_2609_09800_amd import workloads as wl

PAGE = wl.PAGE
BASE = wl.RANGE_BASE
T_READ = 3000
XFER = 2048  # ns per 16 KiB page at 8 GB/s


def _time(name, n, layout, geo, gap=0.0, out=0.0, plane=False, blocking=False, vmem=False):
    c = dict(kind="time", n=n, layout=layout, channels=geo[0], dies=geo[1], planes=geo[2], gap=gap, out=out,
             plane=plane, blocking=blocking, vmem=vmem)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one decode layer's faulted weights: 8 or so matrices of about 192 pages, all issued at once (smallest, latency bound)
        _time("layer_pages", 1536, "pages", (16, 8, 4)),
        # an ordinary open-loop trace: uniform pages and short sequential runs, an odd count
        _time("runs_1m", 1_000_003, "runs", (16, 8, 4), gap=20.0),
        # 16 decode steps of a 64-token batch over the 54 GiB expert set, about 2 us of compute per layer
        _time("moe_decode", 44_500_001, "moe", (16, 8, 4)),
        # the largest stream: MoE weights and a shared KV prefix, 2^28 page reads on 512 dies
        _time("mixed_large", 1 << 28, "mixed", (32, 16, 4), gap=2.0),
        # the same device below saturation: arrivals at 85 % of what its channels carry, so queues stay short
        _time("steady_load", 4_000_001, "mixed", (32, 16, 4), gap=75.0),
        # the same kind of stream where each plane serves its own reads (2,048 die queues, 64 per channel)
        _time("plane_parallel", 3_000_001, "mixed", (32, 16, 4), gap=10.0, plane=True),
        # one page register per die: a die waits for its page's transfer
        _time("register_blocking", 1_000_003, "runs", (16, 8, 4), gap=20.0, blocking=True),
        # closed-loop decode: two steps of 48 layers, each layer issued after the one before completes
        dict(name="closed_loop", kind="layers", steps=2, active=54, compute=2000),
        # a refresh plan handed over and claimed by the reads that follow (73,728 quanta)
        dict(name="refresh", kind="refresh", n=(1 << 25) + 5, gap=2.0, pages_per_block=32),
        # two decode steps of an 8-token batch through a frame cache that holds half of the experts
        dict(name="capacity", kind="capacity", steps=2, active=36, frames=1_769_472, prefetch=7),
        # one layer's grouped GEMV, a batch of 16, nothing faulted: what the instrumented kernel costs by itself
        dict(name="gemv_b16", kind="gemv", experts=8, rows=768, cols=2048, batch=16, faulted=-1),
        # the same layer at a batch of 4 where one of the eight experts is read from HBF and its pages are waited for
        dict(name="paid_layer", kind="gemv", experts=8, rows=768, cols=2048, batch=4, faulted=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    geos = [(8, 4, 1), (16, 8, 4), (32, 16, 4), (16, 8, 4), (32, 16, 4), (12, 5, 2), (64, 8, 2)]
    r = rng.random()
    if r < 0.44:
        layout = rng.choice(["pages", "uniform", "runs", "moe", "mixed", "mixed"])
        geo = rng.choice(geos)
        # mean gap over what one channel page takes of the whole device: below 1 the channels are saturated
        load = rng.choice([rng.uniform(0.02, 0.15), rng.uniform(0.15, 1.0), rng.uniform(1.0, 2.0)])
        hi = {"pages": 1 << 16, "uniform": 1 << 22, "runs": 1 << 22, "moe": 1 << 26, "mixed": 1 << 27 if load < 0.1 else 1 << 23}[layout]
        return _time(None, _log(rng, 1 << 16 if layout == "moe" else 512, hi), layout, geo, gap=round(XFER / geo[0] * load, 1), out=rng.choice([0.0, 0.0, 0.1]))
    if r < 0.50:
        return _time(None, _log(rng, 1024, 1 << 22), rng.choice(["runs", "mixed"]), rng.choice([(16, 8, 4), (32, 16, 4)]),
                     gap=round(rng.uniform(4, 100), 1), plane=True)
    if r < 0.57:
        return _time(None, _log(rng, 1024, 1 << 21), "runs", rng.choice([(16, 8, 4), (32, 16, 4)]),
                     gap=round(rng.uniform(4, 25), 1), blocking=True)
    if r < 0.63:
        return _time(None, _log(rng, 1024, 1 << 26), rng.choice(["moe", "mixed"]), (32, 16, 4),
                     gap=round(rng.uniform(1, 20), 1), vmem=True)
    if r < 0.72:
        return dict(kind="layers", steps=rng.choice([1, 2]), active=rng.randint(8, 54), compute=rng.randint(500, 5000))
    if r < 0.78:
        gap = round(math.exp(rng.uniform(0, math.log(90))), 1)
        return dict(kind="refresh", n=_log(rng, 1 << 18, 1 << 26 if gap < 6 else 1 << 23), gap=gap, pages_per_block=rng.choice([8, 16, 32]))
    if r < 0.85:
        return dict(kind="capacity", steps=rng.choice([1, 2]), active=rng.randint(8, 40),
                    frames=_log(rng, 1_000_000, 2_600_000), prefetch=rng.choice([0, 1, 3, 7, 15, 31, 63]))
    if r < 0.95:
        return dict(kind="gemv", experts=rng.randint(1, 16), rows=16 * rng.randint(4, 96), cols=rng.choice([512, 1024, 2048, 2048, 4096]),
                    batch=rng.choice([1, 1, 2, 4, 5, 8, 12, 16, 24]), faulted=rng.choice([-1, -1, 0, 1]))
    return dict(kind="classify", n=_log(rng, 1 << 16, 1 << 27), channels=32, dies=16, planes=4, ranges=rng.choice([1, 3, 9]))


# ---------------------------------------------------------------- streams

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _poisson(g, n, gap):
    """Issue times: gaps floor(Exponential(gap)) ns, cumulated."""
    if gap <= 0:
        return torch.zeros(n, dtype=torch.int64, device="cuda")
    x = torch.empty(n, dtype=torch.float32, device="cuda").exponential_(1.0 / gap, generator=g)
    return torch.cumsum(x.to(torch.int64), 0)


def _active(active, step, layer):
    """Distinct experts that a layer reads: they vary a little around the batch's usual number."""
    return max(1, active - 2 + (5 * layer + 3 * step) % 5)


class _Router:
    """Zipf(1.1) experts with a fixed permutation per layer, drawn without replacement."""

    def __init__(self, g):
        self.g, self.steps = g, 0
        w = -wl.ZIPF_S * torch.log(torch.arange(1, wl.MOE_EXPERTS + 1, dtype=torch.float32, device="cuda"))
        perm = torch.rand((wl.MOE_LAYERS, wl.MOE_EXPERTS), device="cuda", generator=g).argsort(dim=1)
        self.logw = torch.empty((wl.MOE_LAYERS, wl.MOE_EXPERTS), device="cuda")
        self.logw.scatter_(1, perm, w.expand(wl.MOE_LAYERS, -1).contiguous())

    def step(self, active):
        """(pages in layer order, pages per layer) of one decode step: experts ascending, each one's pages in order."""
        e = torch.empty((wl.MOE_LAYERS, wl.MOE_EXPERTS), device="cuda").exponential_(generator=self.g)
        rank = (torch.log(e) - self.logw).argsort(dim=1).argsort(dim=1)
        size = torch.tensor([_active(active, self.steps, i) for i in range(wl.MOE_LAYERS)], device="cuda")
        self.steps += 1
        first = (rank < size[:, None]).flatten().nonzero().flatten() * wl.PAGES_PER_EXPERT
        pages = (first[:, None] + torch.arange(wl.PAGES_PER_EXPERT, device="cuda")).flatten()
        return pages, size * wl.PAGES_PER_EXPERT


def _decode_pages(case):
    """Pages of a case's decode steps."""
    return wl.PAGES_PER_EXPERT * sum(_active(case["active"], s, i) for s in range(case["steps"]) for i in range(wl.MOE_LAYERS))


def _moe(g, n, active=54):
    """The first n pages of as many decode steps as they take, and the pages of each layer.

    The first pages of each layer, up to an expert's, are still resident and are not read.
    """
    router, pages, sizes, got = _Router(g), [], [], 0
    while got < n:
        pg, sz = router.step(active)
        held = torch.randint(0, wl.PAGES_PER_EXPERT, (sz.numel(),), device="cuda", generator=g)
        first = torch.repeat_interleave(torch.cumsum(sz, 0) - sz + held, sz)
        pg, sz = pg[torch.arange(pg.numel(), device="cuda") >= first], sz - held
        pages.append(pg)
        sizes.append(sz)
        got += pg.numel()
    return torch.cat(pages)[:n], torch.cat(sizes)


def _stream(case, g):
    """(addresses, issue times, range bytes) of a time case."""
    n, layout = case["n"], case["layout"]
    rbytes = 64 * wl.GIB
    issue = None
    if layout == "pages":
        size = torch.randint(128, 257, (n // 128 + 1,), device="cuda", generator=g)
        first = torch.randint(0, rbytes // PAGE - 256, (size.numel(),), device="cuda", generator=g)
        shift = torch.repeat_interleave(first - (torch.cumsum(size, 0) - size), size)[:n]
        pg = shift + torch.arange(n, device="cuda")
        issue = torch.zeros(n, dtype=torch.int64, device="cuda")
    elif layout == "uniform":
        pg = torch.randint(0, rbytes // PAGE, (n,), device="cuda", generator=g)
    elif layout == "runs":
        single = torch.rand(n, device="cuda", generator=g) < 32.0 / 33.0
        run = torch.empty(n, device="cuda").geometric_(1.0 / 32.0, generator=g).clamp_(1, 256).to(torch.int64)
        run[single] = 1
        start = torch.randint(0, rbytes // PAGE, (n,), device="cuda", generator=g)
        end = torch.cumsum(run, 0)
        at = torch.arange(n, device="cuda")
        seg = torch.searchsorted(end, at, right=True)
        pg = (start[seg] + at - (end[seg] - run[seg])) % (rbytes // PAGE)
    elif layout == "moe":
        pg, sizes = _moe(g, n)
        if not case["vmem"]:
            spacing = torch.randint(1500, 2501, (sizes.numel(),), device="cuda", generator=g)
            issue = torch.repeat_interleave(torch.cumsum(spacing, 0) - spacing, sizes)[:n].contiguous()
    else:
        rbytes = wl.TIB
        kv = torch.rand(n, device="cuda", generator=g) < 0.2
        n_kv = int(kv.sum())
        pg = torch.empty(n, dtype=torch.int64, device="cuda")
        pg[~kv] = _moe(g, n - n_kv)[0]
        pg[kv] = 64 * wl.GIB // PAGE + torch.arange(n_kv, device="cuda") % wl.KV_PAGES
        del kv
    addr = pg * PAGE + BASE
    if case.get("out"):
        far = torch.rand(n, device="cuda", generator=g) < case["out"]
        addr[far] += rbytes
    if issue is None:
        issue = _poisson(g, n, case["gap"])
    return addr, issue, rbytes


def _flags(case):
    return (hbf.HBF_FLAG_PLANE_PARALLEL * bool(case.get("plane")) | hbf.HBF_FLAG_REGISTER_BLOCKING * bool(case.get("blocking"))
            | hbf.HBF_FLAG_VMEM_CURVE * bool(case.get("vmem")))


def _model(geo, ranges, flags=0):
    m = hbf.Model(**wl.geometry(*geo, t_read_ns=T_READ, flags=flags))
    for b, n in ranges:
        assert m.register_range(b, n)[0] == 0
    return m


def _refresh_blocks(seed):
    """One block of every plane of the 32 x 16 x 4 device, then one more plane-0 block of half of the dies."""
    r = np.random.Generator(np.random.PCG64(seed))
    blocks = [(0, p % 2, c, d, p, int(r.integers(0, 1024))) for c in range(32) for d in range(16) for p in range(4)]
    return blocks + [(1, 0, int(q) // 16, int(q) % 16, 0, int(r.integers(0, 1024))) for q in np.sort(r.permutation(512)[:256])]


def _class_ranges(case):
    """The ranges of a classify case: equal shares of a tebibyte with gaps of the same size between them."""
    share = wl.TIB // case["ranges"] // PAGE * PAGE
    return [(BASE + 2 * k * share, share) for k in range(case["ranges"])]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "time":
        s["addr"], s["issue"], rbytes = _stream(case, g)
        s["model"] = _model((case["channels"], case["dies"], case["planes"]), [(BASE, rbytes)], _flags(case))
        if case["vmem"]:
            assert s["model"].vmem_configure(wl.VMEM_KNOTS) == 0
        s["complete"] = torch.empty_like(s["issue"])
    elif kind == "layers":
        router, pages, sizes = _Router(g), [], []
        for _ in range(case["steps"]):
            pg, sz = router.step(case["active"])
            pages.append(pg)
            sizes.append(sz)
        s["addr"] = torch.cat(pages) * PAGE + BASE
        s["starts"] = np.concatenate([[0], np.cumsum(torch.cat(sizes).cpu().numpy())]).astype(np.int64)
        s["compute"] = case["compute"]
        s["model"] = _model((16, 8, 4), [(BASE, wl.MOE_LAYERS * wl.MOE_EXPERTS * wl.EXPERT_BYTES)])
        s["issue"] = torch.empty_like(s["addr"])
        s["complete"] = torch.empty_like(s["addr"])
        s["done"] = torch.empty(s["starts"].size - 1, dtype=torch.int64, device="cuda")
    elif kind == "refresh":
        s["addr"], s["issue"], rbytes = _stream(dict(n=case["n"], layout="mixed", gap=case["gap"], vmem=False), g)
        s["model"] = _model((32, 16, 4), [(BASE, rbytes)])
        assert s["model"].refresh_configure(30_000) == 0
        rc, s["pages"] = hbf.refresh_plan(wl.geometry(32, 16, 4), _refresh_blocks(seed), case["pages_per_block"])
        assert rc == 0
        s["complete"] = torch.empty_like(s["issue"])
        s["done"] = torch.empty(s["pages"].size, dtype=torch.int64, device="cuda")
    elif kind == "capacity":
        router = _Router(g)
        s["pages"] = torch.cat([router.step(case["active"])[0] for _ in range(case["steps"])])
        n = s["pages"].numel()
        s["cache"] = hbf.Cache(case["frames"], case["prefetch"], wl.MOE_LAYERS * wl.MOE_EXPERTS * wl.PAGES_PER_EXPERT)
        s["hit"] = torch.zeros(n, dtype=torch.uint8, device="cuda")
        s["counts"] = torch.zeros(8, dtype=torch.int64, device="cuda")
        s["pf_page"] = torch.zeros(n * (2 if case["prefetch"] else 1), dtype=torch.int64, device="cuda")
        s["pf_src"] = torch.zeros_like(s["pf_page"])
    elif kind == "gemv":
        E, N, K, B = case["experts"], case["rows"], case["cols"], case["batch"]
        room = torch.empty(E * N * K + PAGE // 2, dtype=torch.int16, device="cuda")
        off = (-room.data_ptr()) % PAGE // 2
        s["W"] = room[off:off + E * N * K].view(E, N, K)
        w = torch.randn((E, N, K), device="cuda", generator=g) / math.sqrt(K)
        s["W"].copy_(w.to(torch.bfloat16).view(torch.int16))
        s["X"] = torch.randn((E, B, K), device="cuda", generator=g).to(torch.bfloat16).view(torch.int16)
        s["Y"] = torch.empty((E, B, N), dtype=torch.float32, device="cuda")
        s["model"] = _model((16, 8, 4), [(s["W"].data_ptr(), E * N * K * 2)])
        s["issue"] = s["complete"] = None
        if case["faulted"] >= 0:
            # the first experts' pages are read from HBF, the others are resident
            pages = E * N * K * 2 // PAGE
            s["issue"] = torch.zeros(pages, dtype=torch.int64, device="cuda")
            s["complete"] = torch.zeros_like(s["issue"])
            read = min(case["faulted"], E) * pages // E
            if read:
                addr = s["W"].data_ptr() + torch.arange(read, device="cuda") * PAGE
                assert s["model"].time_requests(addr, s["issue"][:read], s["complete"][:read]) == 0
                torch.cuda.synchronize()
    else:
        ranges = _class_ranges(case)
        s["addr"] = torch.randint(BASE - wl.TIB // 16, ranges[-1][0] + ranges[-1][1] + wl.TIB // 16, (case["n"],),
                                  device="cuda", generator=g)
        s["model"] = _model((case["channels"], case["dies"], case["planes"]), ranges)
        s["map"] = torch.empty_like(s["addr"])
    return s


def _ok(rc):
    if rc != 0:
        raise RuntimeError(hbf.strerror(rc))


def run(s):
    kind = s["kind"]
    if kind == "time":
        s["model"].reset()
        _ok(s["model"].time_requests(s["addr"], s["issue"], s["complete"]))
        return s["complete"]
    if kind == "layers":
        s["model"].reset()
        _ok(s["model"].time_layers(s["addr"], s["starts"], 0, s["compute"], s["issue"], s["complete"], s["done"]))
        return [s["issue"], s["complete"], s["done"]]
    if kind == "refresh":
        s["model"].reset()
        _ok(s["model"].refresh_submit(s["pages"], s["done"]))
        _ok(s["model"].time_requests(s["addr"], s["issue"], s["complete"]))
        return [s["complete"], s["done"]]
    if kind == "capacity":
        _ok(s["cache"].reset())
        _ok(s["cache"].access(s["pages"], s["hit"], s["counts"], s["pf_page"], s["pf_src"]))
        return [s["hit"], s["counts"], s["pf_page"], s["pf_src"]]
    if kind == "gemv":
        _ok(s["model"].gemv_instrumented(s["W"], s["X"], s["Y"], s["issue"], s["complete"]))
        return s["Y"]
    _ok(s["model"].classify_map(s["addr"], s["map"]))
    return s["map"]


def work(case):
    kind = case["kind"]
    if kind == "time":  # address and issue time in, completion out
        return dict(bytes=24 * case["n"], flops=0)
    if kind == "layers":  # address in, issue and completion out
        return dict(bytes=24 * _decode_pages(case), flops=0)
    if kind == "refresh":  # a quantum: its page in, its completion out
        return dict(bytes=24 * case["n"] + 16 * 2304 * case["pages_per_block"], flops=0)
    if kind == "capacity":  # page in, hit flag out; a prefetch read: page and source out
        n = _decode_pages(case)
        d = case["prefetch"]
        return dict(bytes=9 * n + 16 * n * d // (d + 1) * 3 // 4, flops=0)
    if kind == "gemv":
        E, N, K, B = case["experts"], case["rows"], case["cols"], case["batch"]
        times = 16 * (E * N * K * 2 // PAGE) if case["faulted"] >= 0 else 0
        return dict(bytes=2 * E * N * K + 2 * E * B * K + 4 * E * B * N + times, flops=2 * E * N * K * B)
    return dict(bytes=16 * case["n"], flops=0)


def tolerance(case):
    # Times, flags, counters and map words are integers with one right value.  The GEMV multiplies bf16 exactly and
    # sums in 32 bits: 2,048 terms in another order differ by a few 1e-7.
    return {"rel": 1e-6, "max": 1e-5} if case["kind"] == "gemv" else "exact"


def _seq_free(issue, service):
    """Departures of one first-come-first-served queue, idle at the start."""
    j = np.arange(issue.size, dtype=np.int64)
    return np.maximum.accumulate(issue - j * service) + (j + 1) * service


def exact(case, seed):
    """The same outputs by plain numpy, where that is quick; the media variants are left out."""
    kind = case["kind"]
    if kind == "gemv":
        s = prepare(case, seed)
        X = s["X"].view(torch.bfloat16).cpu().double()
        W = s["W"].view(torch.bfloat16).cpu().double()
        return torch.stack([X[e] @ W[e].T for e in range(X.shape[0])])
    if kind == "classify" and case["n"] <= 1 << 23:
        addr = prepare(case, seed)["addr"].cpu().numpy()
        out, first = np.zeros_like(addr), 0
        for r, (b, size) in enumerate(_class_ranges(case)):
            p = (addr - b) // PAGE + first
            w = ((p % case["channels"]) << 32) | ((p // case["channels"] % case["dies"]) << 42)
            p = p // case["channels"] // case["dies"]
            w |= ((p % case["planes"]) << 50) | (p // case["planes"]) | (r << 56) | np.int64(-1 << 63)
            out = np.where((addr >= b) & (addr < b + size), w, out)
            first += size // PAGE
        return out
    if kind == "time" and case["n"] <= 1 << 22 and not case["blocking"] and not case["vmem"]:
        C, D, P = case["channels"], case["dies"], case["planes"]
        addr, issue, rbytes = _stream(case, _gen(seed))
        addr, issue = addr.cpu().numpy(), issue.cpu().numpy()
        out = issue.copy()
        at = np.flatnonzero((addr >= BASE) & (addr < BASE + rbytes))
        p = (addr[at] - BASE) // PAGE
        key = p % C * D + p // C % D
        if case["plane"]:
            key = key * P + p // (C * D) % P
        order = np.argsort(key, kind="stable")
        done = np.empty_like(p)
        for q in np.split(order, np.flatnonzero(np.diff(key[order])) + 1):
            done[q] = _seq_free(issue[at[q]], T_READ)
        order = np.lexsort((at, done, p % C))
        for q in np.split(order, np.flatnonzero(np.diff((p % C)[order])) + 1):
            out[at[q]] = _seq_free(done[q], XFER)
        return out
    return None
