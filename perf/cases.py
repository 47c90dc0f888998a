"""The work that a user of this library has it do, as cases that can be timed.

A case is a dict of plain values:

  op        what is called: "file" (Archive.decode_all), "range" (Archive.decode_range),
            "region" (Archive.decode_region), "reads" (Archive.read_lookup), "batch"
            (Archive.decode_batch), "verify" (Archive.verify), "split_file", "split_range",
            "split_reads" (the same calls of SplitArchive), "encode" (encode)
  text      "fastq" (4-line records, 150 bp), "fasta" (a genome of 24 sequences) or "noise"
            (bytes without structure: what is stored rather than compressed)
  bytes     size of the text
  block     log2 of the block size, 14 unless the user chose smaller blocks
  penalty   the encoder's level penalty: 32 gives shallow archives, 0 the deepest ones
  n         reads or requests of one call; length of a range in bytes, of a region in bases

Texts are made on the GPU from the seed alone, encoded with the segmented parse that large inputs
take, and bound; outputs, scratch and request tables are allocated once, as a serving loop does.
"""
import functools
import math
import os

import numpy as np
import torch

import paper_2606_18900_amd as lz

DEV = "cuda" if torch.cuda.is_available() else "cpu"
READ = 150                                # bases of a FASTQ record
LINE = 60                                 # bases of a FASTA line
LARGEST = 256 << 20                       # bytes of the largest text


def listed():
    return [
        # the smallest call: one record of a FASTQ file, a latency
        dict(name="read_one", op="reads", text="fastq", bytes=128 << 20, block=14, penalty=32, n=1),
        # an aligner's or a sampler's batch of records
        dict(name="reads_4096", op="reads", text="fastq", bytes=128 << 20, block=14, penalty=32, n=4096),
        # a serving batch: 90 % records, 10 % byte ranges of 4 KiB to 1 MiB
        dict(name="batch_256", op="batch", text="fastq", bytes=128 << 20, block=14, penalty=32, n=256),
        # chr:start-end of a genome, a small odd size
        dict(name="region_20k", op="region", text="fasta", bytes=64 << 20, block=14, penalty=32, n=20011),
        # one window of a genome that is streamed; the range begins and ends inside blocks
        dict(name="range_window", op="range", text="fasta", bytes=128 << 20, block=14, penalty=32, n=(48 << 20) + 777),
        # a small file: 12,000 records, fewer blocks than the chip has room for
        dict(name="file_small", op="file", text="fastq", bytes=3999999, block=14, penalty=32),
        # whole-file decode, the headline use, on the two kinds of text
        dict(name="file_fastq", op="file", text="fastq", bytes=LARGEST, block=14, penalty=32),
        dict(name="file_genome", op="file", text="fasta", bytes=128 << 20, block=14, penalty=32),
        # an archive written without the level penalty: 64 dependency levels
        dict(name="file_deep", op="file", text="fastq", bytes=64 << 20, block=14, penalty=0),
        # the stream-separated container: four archives, then the records put together
        dict(name="split_file", op="split_file", text="fastq", bytes=64 << 20, block=14, penalty=32),
        # a decoded file checked against its source's hashes
        dict(name="verify", op="verify", text="fastq", bytes=128 << 20, block=14, penalty=32),
        # compression on the host with the default profile: 12,000 records
        dict(name="encode_small", op="encode", text="fastq", bytes=3999999, block=14, penalty=32),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["file", "file", "range", "region", "reads", "reads", "batch", "verify",
                     "split_file", "split_range", "split_reads"])
    c = dict(op=op, text="fastq", bytes=_log(rng, 1 << 20, 128 << 20), block=14, penalty=32)
    if op in ("file", "range", "verify"):
        c["text"] = rng.choice(["fastq", "fastq", "fasta", "fasta", "noise"])
        c["block"] = rng.choice([14, 14, 14, 13, 12])
    if op == "region":
        c["text"] = "fasta"
    if op in ("file", "range", "reads", "batch") and c["text"] == "fastq" and c["bytes"] <= 64 << 20:
        c["penalty"] = rng.choice([32, 32, 0])
    if op in ("range", "split_range"):
        c["n"] = _log(rng, 1000, c["bytes"] // 2)
    if op == "region":
        c["n"] = _log(rng, 100, min(1 << 20, c["bytes"] // 16))
    if op in ("reads", "batch", "split_reads"):
        c["n"] = _log(rng, 1, 4096 if op == "reads" else 512)
    return c


# ---- texts ------------------------------------------------------------------

def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (int(seed) + 1) + what)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _ints(g, lo, hi, shape, dtype=torch.int64):
    return torch.randint(lo, hi, shape, generator=g, device=DEV, dtype=dtype)


def _letters(s):
    return torch.tensor(list(s), dtype=torch.uint8, device=DEV)


def _number(v, out, col, digits):
    for k in range(digits):
        out[:, col + k] = (48 + v // 10 ** (digits - 1 - k) % 10).to(torch.uint8)


def _fastq(nbytes, seed):
    """Records @SYN:run:lane:tile:x:y, 150 bases, '+', 150 qualities, as many as nbytes hold (the same
    size for every seed): bases uniform with N at 0.1 %, 2 % of the reads copy an earlier one with 1 % substitutions,
    qualities walk between Q2 and Q40 and fall along the read."""
    g = _gen(seed, 1)
    n = max(1, nbytes // (28 + 2 * READ + 5))
    codes = _ints(g, 0, 4, (n, READ), torch.uint8)
    rows = torch.nonzero(_rand(g, n) < 0.02).flatten()
    rows = rows[rows > 0]
    src = (_rand(g, rows.numel()) * rows).to(torch.int64)
    sub = _ints(g, 1, 4, (rows.numel(), READ), torch.uint8) * (_rand(g, rows.numel(), READ) < 0.01)
    codes[rows] = (codes[src] + sub) % 4
    codes[_rand(g, n, READ) < 0.001] = 4
    q = torch.empty(n, READ, dtype=torch.uint8, device=DEV)
    cur = _ints(g, 34, 41, (n,)).to(torch.float32)
    fell = torch.zeros(n, dtype=torch.bool, device=DEV)
    for j in range(READ):
        if j:
            mu = 38.0 - 14.0 * ((j - 1) / 149.0) ** 2
            cur = cur + torch.floor(0.25 * (mu - cur) + 0.5) + _ints(g, -2, 3, (n,))
            cur = cur.clamp_(2, 40)
        fell |= _rand(g, n) < 0.002
        cur = torch.where(fell, torch.full_like(cur, 2.0), cur)
        q[:, j] = cur.to(torch.uint8) + 33
    r = torch.arange(n, device=DEV)
    rec = torch.empty(n, 28 + 2 * READ + 5, dtype=torch.uint8, device=DEV)
    rec[:, :17] = _letters(b"@SYN:%04d:0:0000:" % int(_ints(g, 1000, 10000, (1,))[0]))
    _number(1 + 8 * r // n, rec, 10, 1)
    _number(1101 + r // 4000 % 16 + 100 * (r // 64000 % 2), rec, 12, 4)
    keep = torch.ones_like(rec, dtype=torch.bool)
    for col in (17, 23):                  # x and y in [1000, 32767], 28 % of them of 4 digits
        short = torch.randperm(n, generator=g, device=DEV) < n * 9000 // 31768
        v = torch.where(short, _ints(g, 1000, 10000, (n,)), _ints(g, 10000, 32768, (n,)))
        _number(v, rec, col, 5)
        keep[:, col] = ~short
    rec[:, 22] = 58
    rec[:, 28] = 10
    rec[:, 29:29 + READ] = _letters(b"ACGTN")[codes.to(torch.int64)]
    rec[:, 29 + READ:32 + READ] = _letters(b"\n+\n")
    rec[:, 32 + READ:32 + 2 * READ] = q
    rec[:, 32 + 2 * READ] = 10
    ends = torch.cumsum(keep.sum(1), 0).cpu().numpy()
    return rec[keep].cpu().numpy(), np.concatenate([[0], ends]).astype(np.int64)


def _fasta(nbytes, seed):
    """24 sequences of falling length, 60 bases a line: GC 41 %, about 45 % copies of a library of 500
    repeats at 5 to 20 % divergence, 3 % tandem arrays, runs of N at both ends and inside."""
    g = _gen(seed, 2)
    host = np.random.default_rng([int(seed), 2])
    names = [b">chr%s\n" % str(k).encode() for k in list(range(1, 23)) + ["X", "Y"]]
    weight = np.arange(24, 0, -1) / 300.0
    lens = np.maximum(1, (weight * (nbytes - 200) * LINE // (LINE + 1)).astype(np.int64))
    n = int(lens.sum())
    # pool: the repeats, then the tandem units; a feature reads its part of it with a period
    elem = np.exp(host.uniform(math.log(300), math.log(6000), 500)).astype(np.int64)
    zipf = 1.0 / np.arange(1, 501)
    k = n // 1500 + 64
    tandem = host.random(k) < 0.1
    pick = host.choice(500, k, p=zipf / zipf.sum())
    unit = np.exp(host.uniform(math.log(2), math.log(200), k)).astype(np.int64)
    array = np.exp(host.uniform(math.log(50), math.log(5000), k)).astype(np.int64)
    eoff = np.concatenate([[0], np.cumsum(elem)])
    uoff = eoff[-1] + np.concatenate([[0], np.cumsum(unit)])
    size = np.empty(2 * k, np.int64)
    size[0::2] = host.geometric(1.0 / 1972.0, k)
    size[1::2] = np.where(tandem, array, elem[pick])
    at = np.concatenate([[0], np.cumsum(size)])
    base = np.zeros(2 * k, np.int64)
    base[1::2] = np.where(tandem, uoff[:-1], eoff[pick])
    period = np.ones(2 * k, np.int64)
    period[1::2] = np.where(tandem, unit, elem[pick])
    rate = np.zeros(2 * k, np.float32)
    rate[1::2] = np.where(tandem, 0.01, host.uniform(0.05, 0.20, k))

    def background(m):
        u = _rand(g, m)
        return ((u > 0.295).to(torch.uint8) + (u > 0.5) + (u > 0.705)).to(torch.uint8)

    pool = background(int(uoff[-1]))
    seg = torch.repeat_interleave(torch.arange(2 * k, device=DEV), torch.as_tensor(size, device=DEV))[:n]
    dev = [torch.as_tensor(v, device=DEV) for v in (at, base, period, rate)]
    off = torch.arange(seg.numel(), device=DEV) - dev[0][seg]
    code = background(n)
    copied = pool[dev[1][seg] + off % dev[2][seg]]
    sub = _ints(g, 1, 4, (seg.numel(),), torch.uint8) * (_rand(g, seg.numel()) < dev[3][seg])
    code[:seg.numel()] = torch.where((seg & 1).bool(), (copied + sub) % 4, code[:seg.numel()])
    parts, p = [], 0
    for name, length in zip(names, lens.tolist()):
        c = code[p:p + length]
        p += length
        end, mid = min(10000, length // 20), length // 200
        inner = int(host.integers(0, max(1, length - mid)))
        for a, b in ((0, end), (length - end, length), (inner, inner + mid)):
            c[a:b] = 4
        letters = _letters(b"ACGTN")[c.to(torch.int64)]
        full = length // LINE
        body = torch.full((full, LINE + 1), 10, dtype=torch.uint8, device=DEV)
        body[:, :LINE] = letters[:full * LINE].view(full, LINE)
        parts += [_letters(name), body.flatten()]
        if length % LINE:
            parts += [letters[full * LINE:], _letters(b"\n")]
    return torch.cat(parts).cpu().numpy(), None


def _noise(nbytes, seed):
    return _ints(_gen(seed, 3), 0, 256, (nbytes,), torch.uint8).cpu().numpy(), None


def _text(case, seed):
    return {"fastq": _fastq, "fasta": _fasta, "noise": _noise}[case["text"]](case["bytes"], seed)


# ---- requests -----------------------------------------------------------------

def _ids(rng, n_reads, k):
    """Half uniform, half Zipf(1.1) over a permutation: popular records come again."""
    cdf = np.cumsum(np.arange(1, n_reads + 1) ** -1.1)
    zipf = rng.permutation(n_reads)[np.searchsorted(cdf, rng.random(k) * cdf[-1]).clip(0, n_reads - 1)]
    return np.where(rng.random(k) < 0.5, rng.integers(0, n_reads, k), zipf).astype(np.int64)


def _spans(case, starts, total, seed):
    """(kind, a, b) of each request and the bytes [lo, hi) that it asks for. One in ten of a batch is a
    range; their lengths are the quantiles of a length log-uniform in [4 KiB, 1 MiB]."""
    rng = np.random.default_rng([int(seed), 4])
    k = case["n"]
    ids = _ids(rng, len(starts) - 1, k)
    lo, hi = starts[ids], starts[ids + 1]
    ranges = k // 10 if case["op"] == "batch" else 0
    size = np.minimum(_lengths(ranges), total)
    pick = rng.permutation(k)[:ranges]
    lo[pick] = np.minimum(lo[pick], total - size)
    hi[pick] = lo[pick] + size
    ranged = np.zeros(k, bool)
    ranged[pick] = True
    return np.where(ranged, 1, 0), np.where(ranged, lo, ids), np.where(ranged, hi - lo, 0), lo, hi


def _lengths(k):
    return np.exp(math.log(4096) + math.log(256) * (np.arange(k) + 0.5) / max(1, k)).astype(np.int64)


def _capacity(case, total):
    """Bytes that any requests of the case fit in."""
    size = int(np.minimum(_lengths(case["n"] // 10), total).sum()) if case["op"] == "batch" else 0
    return size + case["n"] * (28 + 2 * READ + 5)


def _range(case, total, seed):
    rng = np.random.default_rng([int(seed), 5])
    n = min(case["n"], total)
    return int(rng.integers(0, total - n + 1)), n


def _region(case, seqs, seed):
    rng = np.random.default_rng([int(seed), 6])
    fits = [s for s in range(len(seqs)) if seqs[s] >= case["n"]]
    k = int(rng.choice(fits))
    return k, int(rng.integers(0, seqs[k] - case["n"] + 1))


def _params(case):
    return dict(block_log2=case["block"], level_penalty=case["penalty"], hash_bits=22, chain_depth=16,
                segment_log2=20, threads=_threads())


@functools.lru_cache(None)
def _threads():
    return max(1, min(16, len(os.sched_getaffinity(0))))


# ---- the interface --------------------------------------------------------------

def _warm(arc, split):
    """One range over the whole file, planned by one workgroup, as a serving program does once before
    it takes requests: from then on every table of the handle has been written."""
    out = torch.empty(arc.n, dtype=torch.uint8, device=DEV)
    if split:                                # streams of at most 4096 blocks
        arc.decode_range(0, arc.n, out)
        return
    plan = int(arc.tuning().plan_blocks)
    arc.set_tuning(plan_blocks=1 << 20)
    arc.decode_range(0, arc.n, out)
    arc.set_tuning(plan_blocks=plan)


def prepare(case, seed):
    text, starts = _text(case, seed)
    op = case["op"]
    s = dict(op=op)
    if op == "encode":
        s["text"], s["out"] = text, np.zeros(2 * len(text), np.uint8)
        return s
    kind = {"fastq": 1, "fasta": 2, "noise": 0}[case["text"]]
    split = op.startswith("split")
    if split:
        arc = lz.SplitArchive(lz.encode_split(text, **_params(case)))
    else:
        arc = lz.Archive(lz.encode(text, kind=kind, **_params(case)))
    s["arc"] = arc
    if op not in ("file", "split_file", "verify"):
        _warm(arc, split)
    empty = functools.partial(torch.empty, dtype=torch.uint8, device=DEV)
    if op in ("file", "split_file", "verify"):
        s["out"] = empty(arc.n)
    if op == "verify":
        arc.decode_all(s["out"])
    if op in ("range", "split_range"):
        s["offset"], s["n"] = _range(case, arc.n, seed)
        s["out"], s["scratch"] = empty(s["n"]), empty(arc.scratch_bytes(1))
    if op == "region":
        seqs = lz.fasta_index(text)
        k, s["start"] = _region(case, [int(q.length) for q in seqs], seed)
        s["seq"], s["end"], s["out"] = seqs[k], s["start"] + case["n"], empty(case["n"])
        s["scratch"] = empty(2 * case["n"] + 512 + arc.scratch_bytes(1))
    if op in ("reads", "batch", "split_reads"):
        kinds, a, b, _, _ = _spans(case, starts, len(text), seed)
        s["out"] = torch.zeros(_capacity(case, len(text)), dtype=torch.uint8, device=DEV)
        s["offsets"] = torch.empty(case["n"] + 1, dtype=torch.int64, device=DEV)
        s["scratch"] = empty(arc.scratch_bytes(case["n"]))
        s["ids"] = torch.as_tensor(a, device=DEV)
        if op == "batch":
            s["reqs"] = torch.as_tensor(np.stack([kinds, a, b], 1), device=DEV)
            s["count"] = torch.tensor([case["n"]], dtype=torch.int32, device=DEV)
    return s


def run(s):
    op = s["op"]
    if op == "encode":
        packed = lz.encode(s["text"], kind=1, threads=_threads())
        s["out"][:len(packed)] = np.frombuffer(packed, dtype=np.uint8)
        return s["out"]
    arc = s["arc"]
    if op in ("file", "split_file"):
        return arc.decode_all(s["out"])
    if op == "verify":
        return arc.verify(s["out"])
    if op in ("range", "split_range"):
        return arc.decode_range(s["offset"], s["n"], s["out"], s["scratch"])
    if op == "region":
        return arc.decode_region(s["seq"], s["start"], s["end"], s["out"], s["scratch"])
    if op == "batch":
        arc.decode_batch(s["reqs"], s["count"], s["reqs"].shape[0], s["out"], s["offsets"], s["scratch"])
    else:
        arc.read_lookup(s["ids"], s["out"], s["offsets"], s["scratch"])
    return s["out"], s["offsets"]


def work(case):
    """Compressed bytes in, decoded bytes out. A record needs the block that holds it; what its block
    depends on comes on top and is not counted."""
    op, n, block = case["op"], case["bytes"], 1 << case["block"]
    ratio = {"fastq": 2.2 if op.startswith("split") else 1.9, "fasta": 3.2, "noise": 1.0}[case["text"]]
    if op in ("file", "split_file", "encode"):
        return dict(bytes=n + n / ratio, flops=0)
    if op == "verify":
        return dict(bytes=n + 8, flops=0)
    if op in ("range", "split_range", "region"):
        span = case["n"] * (LINE + 1) / LINE if op == "region" else case["n"]
        return dict(bytes=case["n"] + (span + block) / ratio, flops=0)
    out = _capacity(case, n)
    return dict(bytes=out + min(n, out + case["n"] * block) / ratio, flops=0)


def exact(case, seed):
    """In plain numpy: the text itself, or what was asked of it; for a check, the hash over the blocks' hashes."""
    op = case["op"]
    if op == "encode":
        return None
    text, starts = _text(case, seed)
    if op in ("file", "split_file"):
        return torch.from_numpy(text)
    if op in ("range", "split_range"):
        o, n = _range(case, len(text), seed)
        return torch.from_numpy(text[o:o + n].copy())
    if op == "region":
        seqs, at, k = [], 0, -1
        for line in np.split(text, np.flatnonzero(text == ord(">"))[1:]):
            head = int(np.argmax(line == 10)) + 1
            seqs.append((at + head, line.size - head))
            at += line.size
        body = [text[o:o + m] for o, m in seqs]
        bases = [v[v != 10] for v in body]
        k, start = _region(case, [v.size for v in bases], seed)
        return torch.from_numpy(bases[k][start:start + case["n"]].copy())
    if op == "verify":
        return torch.tensor([_tree(text, 1 << case["block"])])
    _, _, _, lo, hi = _spans(case, starts, len(text), seed)
    data = np.concatenate([text[a:b] for a, b in zip(lo, hi)])
    data = np.pad(data, (0, _capacity(case, len(text)) - data.size))
    return torch.from_numpy(data), torch.from_numpy(np.concatenate([[0], np.cumsum(hi - lo)]))


def _fnv(rows):
    h = np.full(rows.shape[0], 0xCBF29CE484222325, dtype=np.uint64)
    for col in np.ascontiguousarray(rows.T):
        h = (h ^ col) * np.uint64(0x100000001B3)
    return h


def _tree(text, block):
    whole = text[:len(text) // block * block].reshape(-1, block)
    parts = [_fnv(whole[k:k + 16384]) for k in range(0, len(whole), 16384)]
    if len(text) % block:
        parts.append(_fnv(text[None, len(text) // block * block:]))
    hashes = np.concatenate(parts)
    return int(_fnv(hashes.astype("<u8").view(np.uint8)[None, :])[0].view(np.int64))
