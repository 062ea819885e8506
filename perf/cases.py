"""Performance cases of the compressor: what its users have it do, through the
public entry points of `paper_2304_07342_amd.gpulz`.

A case names an operation, the content and the parameters:
  op     compress    one buffer to one LZSS stream
         decompress  one LZSS stream back to its buffer
         entropy     one buffer through LZSS and then the Huffman stage
         unentropy   a Huffman-coded LZSS stream back to the buffer
         serve       one step of the batched server: a batch of buffers is
                     compressed and a batch of streams decompressed
  call   handle      buffers and workspace are kept by the caller, as a
                     pipeline over many inputs keeps them; only enqueues
         whole       the convenience call: allocates, waits for the size and
                     returns a tensor of it
  kind   the content (symbol width S follows from it):
         zipf (1)    text-like bytes, the TPC-H string stand-in
         codes (2)   cuSZ-like quantisation codes with copied runs
         sorted (4)  strictly increasing uint32 indices (TPC-H int32)
         f32 (4)     smooth float32 field with noise (RTM stand-in)
         f64 (8)     the same in float64
  nbytes, C (chunk symbols), W (window symbols), MIN (shortest match),
  policy (0 exact longest match, 1 the paper's single window pass).

Contents follow the recipes of `paper_2304_07342_amd.synth`, drawn on the GPU.
All outputs are bytes and whole numbers.
"""
import math

import numpy as np
import torch

from paper_2304_07342_amd import gpulz

WIDTH = {"zipf": 1, "codes": 2, "sorted": 4, "f32": 4, "f64": 8}
# compressed bytes per input byte, about (LZSS; LZSS then Huffman)
LZ_SHARE = {"zipf": 0.99, "codes": 0.48, "sorted": 1.03, "f32": 1.03, "f64": 1.02}
HUFF_SHARE = {"zipf": 0.75, "codes": 0.34, "sorted": 0.75, "f32": 0.9, "f64": 0.95}
MIB = 1 << 20


def _one(name, op, kind, nbytes, C, W, call="handle", MIN=2, policy=0):
    return {"name": name, "op": op, "call": call, "kind": kind, "nbytes": nbytes, "C": C, "W": W,
            "MIN": MIN, "policy": policy}


def listed():
    return [
        # a short record compressed on its own by a service: latency, with the
        # size read back (2-byte codes, ragged last chunk, library defaults)
        _one("compress-codes-20KB-call", "compress", "codes", 20_002, 2048, 128, call="whole"),
        # one field of quantisation codes, the small benchmark workload
        _one("compress-codes-1MiB", "compress", "codes", MIB, 2048, 128),
        # a text column at the parameters that the autotuner picks for bytes
        _one("compress-zipf-64MiB", "compress", "zipf", 64 * MIB, 4096, 256),
        # the headline workload: a simulation field, nearly all literals
        _one("compress-f32-256MiB", "compress", "f32", 256 * MIB, 4096, 256),
        # doubles of a ragged size (tail bytes and a short last chunk) at the
        # small window that the autotuner picks for literal-heavy data
        _one("compress-f64-100MB", "compress", "f64", 100_000_005, 4096, 32),
        # the paper's own match policy on quantisation codes
        _one("compress-codes-scan-16MiB", "compress", "codes", 16 * MIB, 2048, 128, policy=1),
        # a short record read back on its own: latency
        _one("decompress-codes-64KiB-call", "decompress", "codes", 64 << 10, 2048, 128, call="whole"),
        # the text column read back
        _one("decompress-zipf-64MiB", "decompress", "zipf", 64 * MIB, 4096, 256),
        # the simulation field read back
        _one("decompress-f32-256MiB", "decompress", "f32", 256 * MIB, 4096, 256),
        # archiving quantisation codes: LZSS, then the entropy stage
        _one("entropy-codes-128MiB", "entropy", "codes", 128 * MIB, 2048, 128),
        # and reading the archive back
        _one("unentropy-codes-128MiB", "unentropy", "codes", 128 * MIB, 2048, 128),
        # one step of the batched server: mixed widths and sizes, 70% compress
        {"name": "serve-48", "op": "serve", "requests": 48, "lo": 64 << 10, "hi": 16 * MIB,
         "share": 0.7},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["compress", "compress", "compress", "compress", "decompress", "decompress",
                     "entropy", "unentropy", "serve"])
    if op == "serve":
        lo = _log_uniform(rng, 4 << 10, 256 << 10)
        return {"op": "serve", "requests": rng.randint(8, 48), "lo": lo,
                "hi": _log_uniform(rng, 2 * lo, 16 * MIB), "share": round(rng.uniform(0.5, 0.9), 2)}
    kind = rng.choice(["zipf", "codes"]) if op in ("entropy", "unentropy") else \
        rng.choice(["zipf", "codes", "codes", "sorted", "f32", "f64"])
    policy = 1 if op == "compress" and rng.random() < 0.15 else 0
    call = rng.choice(["handle", "handle", "whole"]) if op in ("compress", "decompress") else "handle"
    top = 16 * MIB if policy else 8 * MIB if call == "whole" else 64 * MIB if kind == "zipf" else 128 * MIB
    nbytes = _log_uniform(rng, 4 << 10, top)
    C = rng.choice([1024, 2048, 4096] if WIDTH[kind] == 8 else [1024, 2048, 4096, 8192])
    c = {"op": op, "call": call, "kind": kind, "nbytes": nbytes, "C": C,
         "W": rng.choice([32, 64, 128, 256]), "MIN": rng.choice([2, 2, 2, 3]), "policy": policy}
    return c


# ---- contents ------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand(m, g, dtype=torch.float64):
    return torch.rand(m, generator=g, device="cuda", dtype=dtype)


def _zipf(m, g):
    p = np.arange(1, 65, dtype=np.float64) ** -1.2
    cdf = np.cumsum(p / p.sum())
    cdf[-1] = 1.0
    edges = torch.from_numpy(cdf).cuda()
    out = torch.empty(m, dtype=torch.uint8, device="cuda")
    for i in range(0, m, 1 << 24):
        k = min(1 << 24, m - i)
        out[i:i + k] = (torch.searchsorted(edges, _rand(k, g), right=True) + 0x20).to(torch.uint8)
    return out


def _codes(m, g):
    """uint16 codes: 512 + a rounded Laplace(0, 2), then 30% of the positions
    overwritten by copied runs of 2 to 32 codes from 1 to 128 back (a run that
    is longer than its offset repeats its period)."""
    n = -(-m // 32) * 32
    u = _rand(n, g) - 0.5
    v = 512 - 2.0 * torch.sign(u) * torch.log1p(-2 * u.abs())
    v = v.round().clamp(0, 1023).to(torch.int32)
    rows = n // 32
    L = torch.randint(2, 33, (rows, 1), generator=g, device="cuda")
    o = torch.randint(1, 129, (rows, 1), generator=g, device="cuda")
    start = (_rand(rows, g)[:, None] * (33 - L)).to(torch.int64)
    dst = torch.arange(rows, device="cuda")[:, None] * 32 + start
    on = (_rand(rows, g)[:, None] < 0.3 * 32 / 17) & (dst >= o)
    k = torch.arange(32, device="cuda")[None, :] - start
    copied = on & (k >= 0) & (k < L)
    at = torch.where(copied, dst - o + k.clamp(min=0) % o, torch.arange(n, device="cuda").view(rows, 32))
    return v[at.view(-1)][:m].to(torch.int16)


def _sorted(m, g):
    gaps = torch.floor(torch.log1p(-_rand(m, g)) / math.log(0.7)).to(torch.int64) + 1
    v = torch.cumsum(gaps, 0) & 0xFFFFFFFF
    return torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32)


def _field(m, g, dtype):
    planes = max(1, -(-m // (512 * 256)))
    host = torch.Generator().manual_seed(int(torch.randint(1 << 30, (1,), generator=g, device="cuda")))
    r = torch.rand(8, 3, generator=host, dtype=torch.float64)
    u = torch.randn(8, 3, generator=host, dtype=torch.float64)
    u /= u.norm(dim=1, keepdim=True)
    x = (torch.arange(planes, device="cuda", dtype=torch.float64) / 512)[:, None, None]
    y = (torch.arange(512, device="cuda", dtype=torch.float64) / 512)[None, :, None]
    z = (torch.arange(256, device="cuda", dtype=torch.float64) / 256)[None, None, :]
    acc = torch.randn(planes, 512, 256, generator=g, device="cuda", dtype=torch.float64) * 1e-3
    for k in range(8):
        a, f, phi = 0.1 + 0.9 * float(r[k, 0]), 1 + 15 * float(r[k, 1]), 2 * math.pi * float(r[k, 2])
        ux, uy, uz = (2 * math.pi * f * float(t) for t in u[k])
        acc += a * torch.sin(ux * x + (uy * y + (uz * z + phi)))
    return ((acc / 1e-4).round() * 1e-4).to(dtype).view(-1)[:m]


def _content(kind, nbytes, seed):
    """nbytes bytes of a content, as a uint8 tensor; the bytes after the last
    whole symbol are the start of one more symbol."""
    g = _generator(seed)
    m = -(-nbytes // WIDTH[kind])
    v = {"zipf": lambda: _zipf(m, g), "codes": lambda: _codes(m, g), "sorted": lambda: _sorted(m, g),
         "f32": lambda: _field(m, g, torch.float32), "f64": lambda: _field(m, g, torch.float64)}[kind]()
    return v.contiguous().view(torch.uint8)[:nbytes].clone()


# ---- states --------------------------------------------------------------------

def _handle(case, nbytes):
    c = gpulz.Compressor(nbytes, WIDTH[case["kind"]], case["C"], case["W"], case["MIN"],
                         policy=case["policy"])
    c.out.zero_()  # so that the bytes after the stream are known, too
    return c


def _stream_of(case, x):
    return gpulz.compress(x, WIDTH[case["kind"]], case["C"], case["W"], case["MIN"],
                          policy=case["policy"]).clone()


class _Decoder:
    """What a program keeps to decode streams of up to these sizes."""

    def __init__(self, in_bytes, out_bytes, ws_bytes):
        self.out = torch.zeros(max(out_bytes, 1), dtype=torch.uint8, device="cuda")
        self.ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda")
        self.meta = torch.zeros(2, dtype=torch.int64, device="cuda")
        self.in_bytes, self.out_bytes, self.ws_bytes = in_bytes, out_bytes, ws_bytes

    def args(self, src):
        return (src.data_ptr(), self.in_bytes, self.out.data_ptr(), self.out_bytes,
                self.meta.data_ptr(), self.meta.data_ptr() + 8, self.ws.data_ptr(), self.ws_bytes,
                torch.cuda.current_stream().cuda_stream)


def _lz_decoder(in_bytes, out_bytes):
    return _Decoder(in_bytes, out_bytes, gpulz.gpulz_decompress_workspace_size(in_bytes))


def _prepare_serve(case, seed):
    # the mix of requests belongs to the case; their contents to the seed
    rng = np.random.Generator(np.random.PCG64([case["requests"], case["lo"], case["hi"]]))
    kinds = {1: ["zipf"], 2: ["codes"], 4: ["sorted", "f32"], 8: ["f64"]}
    pool_bytes = case["hi"] // 8 * 8 + 4096
    pools = {k: _content(k, pool_bytes, seed * 8 + i) for i, k in enumerate(WIDTH)}
    comp, dec = [], []
    for r in range(case["requests"]):
        S = int(rng.choice([1, 2, 4, 8]))
        kind = kinds[S][int(rng.integers(len(kinds[S])))]
        n = int(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))) // S * S
        off = int(rng.integers(0, pool_bytes - n + 1)) // 16 * 16
        # the first request compresses and the second decompresses, whatever the share
        first = r == 0 or (r > 1 and rng.random() < case["share"])
        (comp if first else dec).append((pools[kind][off:off + n], S))
    bc = gpulz.BatchCompressor([x for x, _ in comp], [S for _, S in comp])
    for o in bc.outputs:
        o.zero_()
    made = gpulz.BatchCompressor([x for x, _ in dec], [S for _, S in dec])
    made.run()
    streams = [s.clone() for _, s in made.results()]
    bd = gpulz.BatchDecompressor(streams, [x.numel() for x, _ in dec])
    return {"op": "serve", "pools": pools, "compress": bc, "decompress": bd}


def prepare(case, seed):
    if case["op"] == "serve":
        return _prepare_serve(case, seed)
    x = _content(case["kind"], case["nbytes"], seed)
    s = dict(case)
    if case["op"] == "compress":
        s["x"] = x
        if case["call"] == "handle":
            s["handle"] = _handle(case, x.numel())
        else:
            s["record"] = torch.zeros(gpulz.gpulz_compress_bound(x.numel(), WIDTH[case["kind"]], case["C"],
                                                                 case["MIN"]), dtype=torch.uint8, device="cuda")
    elif case["op"] == "entropy":
        s["x"], s["handle"] = x, _handle(case, x.numel())
        s["huff"] = gpulz.HuffCompressor(s["handle"].capacity)
        s["huff"].out.zero_()
    elif case["op"] == "decompress":
        s["stream"] = _stream_of(case, x)
        if case["call"] == "handle":
            s["decoder"] = _lz_decoder(s["stream"].numel(), x.numel())
    else:
        lz = _stream_of(case, x)
        s["stream"] = gpulz.huff_compress(lz).clone()
        s["huff"] = _Decoder(s["stream"].numel(), lz.numel(),
                             gpulz.gpulz_huff_decompress_workspace_size(s["stream"].numel()))
        s["decoder"] = _lz_decoder(lz.numel(), x.numel())
    return s


def _ok(status):
    if status != gpulz.GPULZ_OK:
        raise gpulz.GpulzError(status, "performance case")


def run(state):
    op = state["op"]
    if op == "serve":
        bc, bd = state["compress"], state["decompress"]
        bc.run()
        bd.run()
        return {"streams": bc.outputs, "stream_bytes": bc.d_out_bytes, "status": bc.d_status,
                "buffers": bd.outputs, "buffer_bytes": bd.d_out_bytes, "decode_status": bd.d_status}
    if op == "compress":
        if state["call"] == "whole":
            s = gpulz.compress(state["x"], WIDTH[state["kind"]], state["C"], state["W"],
                               state["MIN"], policy=state["policy"])
            state["record"][:s.numel()] = s  # into the record that the service sends
            return [state["record"], s.numel()]
        h = state["handle"]
        h.compress_async(state["x"])
        return [h.out, h.meta]
    if op == "decompress":
        if state["call"] == "whole":
            return gpulz.decompress(state["stream"])
        d = state["decoder"]
        _ok(gpulz.gpulz_decompress(*d.args(state["stream"])))
        return [d.out, d.meta]
    if op == "entropy":
        h, hc = state["handle"], state["huff"]
        h.compress_async(state["x"])
        hc.compress_async(h.out.data_ptr(), h.capacity, d_nbytes=h.meta.data_ptr())
        return [hc.out, hc.meta, h.meta]
    hd, d = state["huff"], state["decoder"]
    _ok(gpulz.gpulz_huff_decompress(*hd.args(state["stream"])))
    _ok(gpulz.gpulz_decompress(*d.args(hd.out)))
    return [d.out, d.meta, hd.meta]


def work(case):
    if case["op"] == "serve":
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
        share = sum(LZ_SHARE[k] * w for k, w in
                    (("zipf", 2), ("codes", 2), ("sorted", 1), ("f32", 1), ("f64", 2))) / 8
        return {"bytes": int(case["requests"] * mean * (1 + share)), "flops": 0}
    share = (HUFF_SHARE if case["op"] in ("entropy", "unentropy") else LZ_SHARE)[case["kind"]]
    return {"bytes": int(case["nbytes"] * (1 + share)), "flops": 0}
