"""The calls that this library is timed on: what they stand for, their inputs and what one pass of each returns.

A case is a dict of plain values; "kind" picks the entry point:

  align    mica.align on one batch (HIP graph launch, the program's own output buffers)
  noalloc  mica.align_noalloc, the allocation-free call of tight loops
  packed   reads that arrive as base codes on the GPU: mica.pack_2bit, then mica.align
  search   FmIndex.search, the few-mismatch phase
  serve    a burst of requests through a Server: submit, poll, fetch
  pipe     Pipeline.run, FASTQ file in, SAM file out

Reads are simulated the way the benchmark workloads are (a copy of a reference stretch with substitutions and
indels of geometric length, some reads or tails random), drawn on the GPU with torch so that new inputs are cheap.
A reference, an index, a server and a context are things a program keeps for its whole life; they are made once per
process and shared, the reads and windows are new for every seed.
"""
import functools
import os
import tempfile
import time

import numpy as np
import torch

import paper_1402_4876_amd as mica

MODES = {"sg": mica.MODE_SEMIGLOBAL, "local": mica.MODE_LOCAL, "ext": mica.MODE_EXTEND}
DEFAULT = {"match": 1, "mismatch": -4, "open": 6, "extend": 1}


def _align(name, pairs, m_lo, m_hi, win, mode, **more):
    c = {"name": name, "kind": "align", "pairs": pairs, "m_lo": m_lo, "m_hi": m_hi, "win": win, "mode": mode,
         "out": "cigar", "cap": 64, "sub": 0.01, "indel": 0.003, "junk": 0.0, "int32": False, "ref": 100_000_000}
    c.update(DEFAULT)
    c.update(more)
    return c


def listed():
    return [
        # one template's candidate windows inside somebody else's loop: nothing but latency and launches
        _align("align_tiny", 48, 76, 151, 0, "sg", ref=1_000_000),
        # the small 32-bit configuration: 1,000 reads of 150 in windows of 200, scores and end cells only
        _align("align_small_int32", 1000, 150, 150, 200, "sg", out="score", int32=True, indel=0.002, ref=1_000_000),
        # a served batch's mix of read lengths in a loop that may not allocate
        _align("noalloc_batch", 17_000, 100, 250, 0, "sg", kind="noalloc"),
        # the headline workload: a million 150-base reads in 400-base windows, with CIGARs
        _align("align_sg", 1_000_000, 150, 150, 400, "sg"),
        # mate rescue: local alignment in 1,000-base windows, a tenth of the partners unrelated
        _align("align_local", 500_000, 150, 150, 1000, "local", sub=0.02, indel=0.005, junk=0.1),
        # trimmed reads of every length, half of them local
        _align("align_mixed", 1_000_000, 50, 250, 0, "mixed"),
        # seed extension: tails of 0..150 bases after an exact hit, a fifth of them turning random
        _align("align_ext", 1_000_000, 0, 150, 0, "ext", junk=0.2, clip=5),
        # long and noisier reads, another common scoring: the wide plans
        _align("align_long", 12_000, 301, 1000, 0, "sg", sub=0.03, indel=0.01, match=2, mismatch=-4, open=4, extend=2,
               cap=128),
        # ranking candidates by score: odd lengths, codes packed on the GPU first, no traceback
        _align("packed_score", 300_000, 101, 101, 333, "local", kind="packed", out="score", junk=0.3),
        # phase one: a million reads against the whole reference with up to two mismatches
        {"name": "search", "kind": "search", "reads": 1_000_000, "m_lo": 150, "m_hi": 150, "k": 2, "max_occ": 64,
         "sub": 0.01, "indel": 0.003, "ref": 32_000_000},
        # a burst of requests at the server: host staging, copies, small batches in flight
        {"name": "serve_burst", "kind": "serve", "requests": 40, "max_reads": 4000, "sub": 0.01, "indel": 0.003,
         "ref": 256_000_000},
        # the whole product: FASTQ to SAM through both phases
        {"name": "pipeline", "kind": "pipe", "reads": 200_000, "m": 150, "k": 2, "sub": 0.01, "indel": 0.003,
         "ref": 8_000_000},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["align"] * 6 + ["noalloc", "packed", "search", "search", "serve", "pipe"])
    if kind == "search":
        m = rng.randint(36, 250)
        return {"kind": kind, "reads": _log(rng, 1000, 600_000), "m_lo": max(30, m - rng.choice([0, 0, 25])), "m_hi": m,
                "k": rng.randint(0, 2), "max_occ": rng.choice([8, 64, 500]), "sub": 0.01, "indel": 0.003,
                "ref": rng.choice([2_000_003, 12_000_000, 32_000_000])}
    if kind == "serve":
        return {"kind": kind, "requests": rng.randint(1, 40), "max_reads": _log(rng, 10, 4000), "sub": 0.01,
                "indel": 0.003, "ref": 256_000_000}
    if kind == "pipe":
        return {"kind": kind, "reads": _log(rng, 500, 200_000), "m": rng.randint(50, 250), "k": rng.randint(1, 2),
                "sub": 0.01, "indel": 0.003, "ref": 8_000_000}
    m_hi = rng.choice([rng.randint(30, 160), rng.randint(100, 256), rng.randint(257, 1024)])
    m_lo = rng.choice([m_hi, m_hi, max(1, m_hi // 2), max(1, m_hi // 5)])
    win = rng.choice([0, 0, m_hi + rng.randint(10, 400), rng.randint(m_hi, 3 * m_hi)])
    mode = rng.choice(["sg", "local", "mixed", "ext"])
    if mode == "ext":
        win = 0
    n = win or m_hi + (32 if mode == "ext" else m_hi // 2 + 64)
    # no drawn batch computes more cells than the headline one
    pairs = _log(rng, 20, max(40, min(1_000_000, 30_000_000_000 // (m_hi * n))))
    match, mismatch, gap_open, extend = rng.choice([(1, -4, 6, 1), (1, -4, 6, 1), (2, -4, 4, 2), (1, -3, 5, 2)])
    c = _align("", pairs, m_lo, m_hi, win, mode, kind=kind, sub=rng.choice([0.0, 0.005, 0.01, 0.02, 0.05]),
               indel=rng.choice([0.0, 0.002, 0.003, 0.01]), junk=rng.choice([0.0, 0.0, 0.1, 0.3, 1.0]),
               out=rng.choice(["cigar", "cigar", "start", "score"]), cap=rng.choice([16, 64]),
               int32=rng.random() < 0.15, match=match, mismatch=mismatch, open=gap_open, extend=extend,
               ref=rng.choice([1_000_003, 100_000_000]))
    del c["name"]
    if mode == "ext":
        c["clip"] = rng.choice([0, 5, 16])
    if kind == "noalloc":
        c["pairs"] = min(pairs, 100_000)
    return c


# ---- inputs --------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _pack(codes):
    """Codes to 2-bit words (16 bases per int32)."""
    n = codes.numel()
    if n % 16:
        codes = torch.nn.functional.pad(codes, (0, 16 - n % 16))
    shift = torch.arange(0, 32, 2, device=codes.device)
    out = []
    for part in codes.view(-1, 16).split(1 << 22):
        w = (part.to(torch.int64) << shift).sum(1)
        out.append(torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32))
    return torch.cat(out)


@functools.lru_cache(maxsize=None)
def _reference(n):
    """A fixed random genome of n bases: codes, and words with a padding word."""
    codes = torch.randint(0, 4, (n,), dtype=torch.uint8, device="cuda", generator=_gen(14024876 + n))
    return codes, _pack(codes)


@functools.lru_cache(maxsize=None)
def _host_words(n):
    return _reference(n)[1].cpu().numpy().view(np.uint32)


@functools.lru_cache(maxsize=None)
def _context():
    return mica.Context()


@functools.lru_cache(maxsize=None)
def _index(n):
    return mica.FmIndex(_host_words(n), n)


@functools.lru_cache(maxsize=None)
def _server(n):
    return mica.Server(_host_words(n), n, slots=4)


@functools.lru_cache(maxsize=None)
def _pipeline(n, k):
    return mica.Pipeline(_host_words(n), n, "chr1", k=k, batch_reads=65_536)


def _simulate(g, ref, start, width, sub, indel):
    """width read bases for every start: reference bases with substitutions, deletions and random insertions."""
    out = []
    for s in start.split(200_000):
        shape = (s.numel(), width)
        idx = torch.arange(width, device="cuda")
        u = torch.rand(shape, device="cuda", generator=g)
        length = 1 + torch.floor(-torch.log2(1 - torch.rand(shape, device="cuda", generator=g))).to(torch.int64)
        ends = torch.where((u >= indel / 2) & (u < indel), idx + length, 0)
        inside = idx < torch.cummax(ends, 1).values
        step = torch.where(inside, 0, 1 + torch.where(u < indel / 2, length, 0))
        pos = s[:, None] + torch.cumsum(step, 1) - 1
        base = ref[pos.clamp_(0, ref.numel() - 1)]
        other = torch.randint(1, 4, shape, device="cuda", generator=g, dtype=torch.uint8)
        swap = torch.rand(shape, device="cuda", generator=g) < sub
        base = torch.where(swap, (base + other) & 3, base)
        out.append(torch.where(inside, (base + other) & 3, base))
    return torch.cat(out)


def _lay_out(codes, m):
    """Reads one after another, each from a multiple of 16 bases on: (flat codes, offsets)."""
    off = torch.cumsum((m + 15) // 16 * 16, 0)
    total = int(off[-1])
    off = torch.cat([off.new_zeros(1), off[:-1]])
    flat = torch.zeros(max(total, 16), dtype=torch.uint8, device="cuda")
    idx = torch.arange(codes.shape[1], device="cuda")
    for i in range(0, len(m), 200_000):
        keep = idx < m[i:i + 200_000, None]
        flat[(off[i:i + 200_000, None] + idx)[keep]] = codes[i:i + 200_000][keep]
    return flat, off


def _lengths(g, lo, hi, n):
    return torch.randint(lo, hi + 1, (n,), device="cuda", generator=g)


def _window(case, m):
    if case["win"]:
        return torch.full_like(m, case["win"])
    return m + 32 if case["mode"] == "ext" else m * 3 // 2 + 64


def _buffers(case, n):
    """Output tensors that the program keeps."""
    keys = ["score", "read_end", "ref_end", "status"]
    keys += ["read_start", "ref_start"] if case["out"] != "score" else []
    keys += ["n_cigar"] if case["out"] == "cigar" else []
    out = {k: torch.zeros(n, dtype=torch.int32, device="cuda") for k in keys}
    if case["out"] == "cigar":
        out["cigar"] = torch.zeros((n, case["cap"]), dtype=torch.int32, device="cuda")
    return out


def _prepare_align(case, seed):
    g = _gen(seed)
    n, mode = case["pairs"], case["mode"]
    ref, words = _reference(case["ref"])
    m = _lengths(g, case["m_lo"], case["m_hi"], n)
    win = _window(case, m)
    wo = (torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * (case["ref"] - win + 1)).to(torch.int64)
    room = (win - m - 8).clamp(min=0)
    lead = (torch.rand(n, device="cuda", generator=g) * (room + 1)).to(torch.int64) if mode != "ext" else 0
    codes = _simulate(g, ref, wo + lead, case["m_hi"], case["sub"], case["indel"])
    if case["junk"]:
        # whole reads, or for extensions the tail from a random point on
        turn = torch.where(torch.rand(n, device="cuda", generator=g) < case["junk"],
                           (torch.rand(n, device="cuda", generator=g) * m).to(torch.int64) if mode == "ext" else 0 * m,
                           case["m_hi"])
        noise = torch.randint(0, 4, codes.shape, dtype=torch.uint8, device="cuda", generator=g)
        codes = torch.where(torch.arange(case["m_hi"], device="cuda") < turn[:, None], codes, noise)
    flat, ro = _lay_out(codes, m)
    kw = {"scoring": (case["match"], case["mismatch"], case["open"], case["extend"]),
          "out_start": case["out"] == "start", "out_cigar": case["out"] == "cigar", "cigar_cap": case["cap"],
          "force_int32": case["int32"], "max_read_len": case["m_hi"], "min_read_len": case["m_lo"],
          "max_win_len": int(win.max()), "ref_len": case["ref"], "reads_len": flat.numel(), "out": _buffers(case, n)}
    if mode == "mixed":
        kw["mode"] = (torch.rand(n, device="cuda", generator=g) < 0.5).to(torch.uint8)
        kw["mode_mask"] = 3
    else:
        kw["default_mode"] = MODES[mode]
    if mode == "ext":
        kw["ext_h0"] = (torch.randint(19, 61, (n,), device="cuda", generator=g) * case["match"]).to(torch.int32)
        kw["ext_clip"] = case["clip"]
        kw["max_ext_h0"] = 60 * case["match"]
    state = {"kind": case["kind"], "codes": flat, "args": (words, wo, win.to(torch.int32)), "kw": kw,
             "reads": (ro, m.to(torch.int32))}
    if case["kind"] != "packed":
        state["words"] = _pack(flat)
    if case["kind"] != "noalloc":
        state["ctx"] = _context()
    return state


def _prepare_search(case, seed):
    g = _gen(seed)
    n = case["reads"]
    ref, _ = _reference(case["ref"])
    m = _lengths(g, case["m_lo"], case["m_hi"], n)
    start = (torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * (case["ref"] - m - 40)).to(torch.int64)
    flat, ro = _lay_out(_simulate(g, ref, start, case["m_hi"], case["sub"], case["indel"]), m)
    out = {k: torch.zeros(n, dtype=torch.int32, device="cuda") for k in ("best_mm", "n_best", "n_hits", "status")}
    out["pos"] = torch.zeros(n, dtype=torch.int64, device="cuda")
    return {"kind": "search", "index": _index(case["ref"]), "words": _pack(flat), "reads": (ro, m.to(torch.int32)),
            "kw": {"k": case["k"], "max_occ": case["max_occ"], "reads_len": flat.numel(), "out": out}}


def _prepare_serve(case, seed):
    g = _gen(seed)
    ref, _ = _reference(case["ref"])
    # request sizes belong to the case: the same for every seed
    count = np.random.default_rng(case["requests"]).integers(1, case["max_reads"] + 1, case["requests"])
    n = int(count.sum())
    m = torch.tensor([100, 150, 250], device="cuda")[torch.randint(0, 3, (n,), device="cuda", generator=g)]
    win = m * 3 // 2 + 64
    wo = (torch.rand(n, device="cuda", generator=g, dtype=torch.float64) * (case["ref"] - win + 1)).to(torch.int64)
    lead = (torch.rand(n, device="cuda", generator=g) * (win - m - 7)).to(torch.int64)
    flat, ro = _lay_out(_simulate(g, ref, wo + lead, 250, case["sub"], case["indel"]), m)
    keys = ("score", "read_start", "read_end", "ref_start", "ref_end", "n_cigar", "status")
    out = {k: np.zeros(n, np.int32) for k in keys}
    out["cigar"] = np.zeros((n, 64), np.uint32)
    host = [_pack(flat).cpu().numpy().view(np.uint32), ro.cpu().numpy().astype(np.uint64),
            m.cpu().numpy().astype(np.int32), wo.cpu().numpy().astype(np.uint64), win.cpu().numpy().astype(np.int32)]
    first = np.concatenate([[0], np.cumsum(count)])
    return {"kind": "serve", "server": _server(case["ref"]), "host": host, "first": first, "out": out}


def _prepare_pipe(case, seed):
    g = _gen(seed)
    ref, _ = _reference(case["ref"])
    n, m = case["reads"], case["m"]
    start = torch.randint(0, case["ref"] - m - 40, (n,), device="cuda", generator=g)
    codes = _simulate(g, ref, start, m, case["sub"], case["indel"])
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")[codes.long()].cpu().numpy()
    qual = torch.randint(35, 74, (n, m), dtype=torch.uint8, device="cuda", generator=g).cpu().numpy()
    name = np.frombuffer("".join("@read%08d\n" % i for i in range(n)).encode(), np.uint8).reshape(n, -1)
    line = lambda text: np.broadcast_to(np.frombuffer(text, np.uint8), (n, len(text)))  # noqa: E731
    records = np.concatenate([name, letters, line(b"\n+\n"), qual, line(b"\n")], 1)
    folder = tempfile.TemporaryDirectory()
    fastq = os.path.join(folder.name, "reads.fq")
    records.tofile(fastq)
    return {"kind": "pipe", "pipe": _pipeline(case["ref"], case["k"]), "folder": folder, "fastq": fastq,
            "sam": os.path.join(folder.name, "out.sam"), "room": n * (2 * m + 160) + 4096}


def prepare(case, seed):
    make = {"search": _prepare_search, "serve": _prepare_serve, "pipe": _prepare_pipe}.get(case["kind"], _prepare_align)
    return make(case, seed)


# ---- one pass ------------------------------------------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "search":
        return state["index"].search(state["words"], *state["reads"], **state["kw"])
    if kind == "serve":
        return _serve(state)
    if kind == "pipe":
        state["pipe"].run(state["fastq"], state["sam"])
        # records differ in length: zeros to a common size (a hole in the file), mapped rather than read
        os.truncate(state["sam"], state["room"])
        return np.memmap(state["sam"], np.uint8, "r")
    words = mica.pack_2bit(state["codes"]) if kind == "packed" else state["words"]
    if kind == "noalloc":
        return mica.align_noalloc(*state["args"], words, *state["reads"], **state["kw"])
    return mica.align(state["ctx"], *state["args"], words, *state["reads"], **state["kw"])


def _serve(state):
    server, first, out = state["server"], state["first"], state["out"]
    words, ro, m, wo, win = state["host"]
    for r in range(len(first) - 1):
        s = slice(first[r], first[r + 1])
        server.submit(r, words, ro[s], m[s], wo[s], win[s])
    left = len(first) - 1
    while left:
        for r in server.poll():
            server.fetch(r, out={k: v[first[r]:first[r + 1]] for k, v in out.items()})
            left -= 1
        if left:
            time.sleep(20e-6)
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def work(case):
    """Bytes: sequences (2 bits a base), descriptors and results once.  Operations: integer operations of the whole DP
    table, the way cell updates are counted (a method that proves cells irrelevant computes fewer); none for the
    search, which compares and looks up."""
    kind = case["kind"]
    if kind == "search":
        return {"bytes": case["reads"] * (case["m_hi"] / 4 + 12 + 24), "flops": 0}
    if kind == "serve":
        n = case["requests"] * (1 + case["max_reads"]) / 2
        return {"bytes": n * (167 / 4 + 314 / 4 + 25 + 36), "flops": n * 167 * 314 * 13}
    if kind == "pipe":
        return {"bytes": case["reads"] * (4 * case["m"] + 60.0), "flops": 0}
    m = (case["m_lo"] + case["m_hi"]) / 2
    n = case["win"] or (m + 32 if case["mode"] == "ext" else 1.5 * m + 64)
    traced = case["out"] != "score"
    ops = {"sg": 13 if traced else 9, "mixed": 14.5 if traced else 10}.get(case["mode"], 16 if traced else 11)
    per_pair = m / 4 + n / 4 + 25 + 16 + (8 if traced else 0) + (8 if case["out"] == "cigar" else 0)
    if kind == "packed":
        per_pair += 1.25 * m
    return {"bytes": case["pairs"] * per_pair, "flops": case["pairs"] * m * n * ops}


def exact(case, seed):
    """None: every output is a whole number (or a byte of text), held to equality; none is a rounded value."""
    return None
