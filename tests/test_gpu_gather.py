"""Requested bytes copied out of scratch slots: every alignment of source and
destination, lengths around the 16-byte units, the 4 KiB parts and the block
edges, and batches of mixed sizes.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[14, 12, 6])
def arc(request, orc):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, starts = fastq(n_records=400 if request.param > 6 else 40, seed=9)
    a = orc.encode(x, kind=1, block_log2=request.param, level_penalty=32)
    return x, starts, lz.Archive(a)


@pytest.mark.parametrize("shift", [0, 1, 15])
def test_ranges(arc, shift):
    x, _, A = arc
    B = 1 << int(A.info.block_log2)
    for o in (0, 1, 15, 16, B - 1, B, B + 7):
        for n in (1, 15, 16, 17, 31, 4095, 4097, B - 1, B, B + 1, 2 * B + 5):
            n = min(n, len(x) - o)
            buf = torch.full((n + shift + 32,), 7, dtype=torch.uint8, device="cuda")
            A.decode_range(o, n, out=buf[shift:])
            A.sync_status()
            got = buf.cpu().numpy()
            assert got[shift:shift + n].tobytes() == x[o:o + n], (o, n)
            assert (got[:shift] == 7).all() and (got[shift + n:] == 7).all(), (o, n)


def test_batch(arc):
    x, starts, A = arc
    rng = np.random.default_rng(4)
    n = 300
    kind = (rng.random(n) < 0.3).astype(np.int64)
    ids = rng.integers(0, len(starts) - 1, n)
    off = rng.integers(0, len(x), n)
    ln = np.minimum((np.exp(rng.random(n) * 10)).astype(np.int64) - 1, len(x) - off)
    reqs = np.stack([kind, np.where(kind == 1, off, ids), np.where(kind == 1, ln, 0)], 1)
    want = [x[int(a):int(a + b)] if k else x[int(starts[a]):int(starts[a + 1])] for k, a, b in reqs]
    total = sum(map(len, want))
    out = torch.full((total + 64,), 7, dtype=torch.uint8, device="cuda")
    offs = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    scr = torch.empty(A.scratch_bytes(n), dtype=torch.uint8, device="cuda")
    A.decode_batch(torch.as_tensor(reqs, device="cuda"), torch.tensor([n], dtype=torch.int32, device="cuda"),
                   n, out, offs, scr)
    A.sync_status()
    assert int(offs[-1]) == total
    got = out.cpu().numpy()
    assert got[:total].tobytes() == b"".join(want)
    assert (got[total:] == 7).all()
