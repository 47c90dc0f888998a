"""Batches on archives of 256 blocks and more, which a wave copies a part of a
block at a time (test_gpu_gather.py's batches are on smaller ones, which one
workgroup copies), and reads at the limit of one-workgroup planning.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[14, 12])
def wide(request):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, starts = fastq(n_records=14000 if request.param == 14 else 4000, seed=10)
    A = lz.Archive(lz.encode(x, kind=1, block_log2=request.param, level_penalty=32))
    assert A.n_blocks >= 256                   # fewer are gathered by one workgroup
    return x, starts.astype(np.int64), A


def _wide_requests(x, starts, B, rng):
    """Empty ranges, ranges that begin and end on, before and behind the edges
    of parts (a quarter of a block) and of blocks, over up to five blocks, and
    reads, in any order."""
    P, q = B // 4, []
    for base in (0, 3 * B, 100 * B, len(x) - 6 * B):
        for o in (0, 1, P - 1, P, P + 1, B - 17, B - 1):
            for e in (0, 1, 15, 16, 17, P - 1, P, P + 1, 2 * P + 5, B, B + P + 3, 3 * B + 1, 5 * B):
                q.append((1, base + o, e))
    q += [(0, int(r), 0) for r in rng.integers(0, len(starts) - 1, 200)]
    q.append((1, len(x), 0))
    return np.array(q, np.int64)[rng.permutation(len(q))]


@pytest.mark.parametrize("shift,slack", [(0, 64), (5, 64), (0, 80 << 20)])
def test_batch_parts(wide, shift, slack):
    """slack: an output of 80 MiB more is planned by the eight kernels."""
    x, starts, A = wide
    q = _wide_requests(x, starts, 1 << int(A.info.block_log2), np.random.default_rng(shift))
    n = len(q)
    want = [x[a:a + b] if k else x[starts[a]:starts[a + 1]] for k, a, b in q.tolist()]
    ends = np.cumsum([0] + [len(w) for w in want])
    buf = torch.full((shift + int(ends[-1]) + slack,), 7, dtype=torch.uint8, device="cuda")
    offs = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    scr = torch.full((A.scratch_bytes(n),), 0xAA, dtype=torch.uint8, device="cuda")
    A.decode_batch(torch.as_tensor(q, device="cuda"), torch.tensor([n], dtype=torch.int32, device="cuda"),
                   n, buf[shift:], offs, scr)
    A.sync_status()
    assert np.array_equal(offs.cpu().numpy(), ends)
    got = buf[:shift + int(ends[-1]) + 64].cpu().numpy()
    assert got[shift:shift + ends[-1]].tobytes() == b"".join(want)
    assert (got[:shift] == 7).all() and (got[shift + ends[-1]:] == 7).all()


@pytest.mark.parametrize("n", [4096, 4097])
def test_reads_at_the_planner_limit(wide, n):
    """The most reads that one workgroup plans by default, and one more."""
    x, starts, A = wide
    ids = np.random.default_rng(n).integers(0, len(starts) - 1, n)
    got, offs = A.read_lookup(ids)
    A.sync_status()
    want = b"".join(x[starts[r]:starts[r + 1]] for r in ids)
    assert int(offs[-1]) == len(want) and got[:len(want)].cpu().numpy().tobytes() == want
