"""Planning of request calls: one workgroup with its marks and list in LDS, in
LDS as far as it fits (more than 6144 blocks in the closure), with marks in
memory (more than 2^18 blocks), and the eight-kernel path, must give the same
bytes, offsets and closures.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=[(14, 3000), (8, 8000), (6, 55000)])
def arc(request):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    bl, recs = request.param
    x, starts = fastq(n_records=recs, seed=13)
    a = lz.encode(x, kind=1, block_log2=bl, level_penalty=1, hash_bits=22, segment_log2=20)
    return x, starts.astype(np.int64), lz.Archive(a)


@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1025, 4096])
def test_reads_and_batches(arc, n):
    x, starts, A = arc
    if (1 << int(A.info.block_log2)) == 64:
        assert A.n_blocks > 1 << 18
    rng = np.random.default_rng(n)
    nr = len(starts) - 1
    ids = rng.integers(0, nr, n)
    kind = (rng.random(n) < 0.2).astype(np.int64)
    off = rng.integers(0, len(x), n)
    ln = np.minimum(np.exp(rng.random(n) * 9).astype(np.int64) - 1, len(x) - off)
    reqs = np.stack([kind, np.where(kind == 1, off, ids), np.where(kind == 1, ln, 0)], 1)
    want_r = b"".join(x[starts[i]:starts[i + 1]] for i in ids)
    want_b = b"".join(x[a:a + b] if k else x[starts[a]:starts[a + 1]] for k, a, b in reqs)
    d_ids = torch.as_tensor(ids, device="cuda")
    d_reqs = torch.as_tensor(reqs, device="cuda")
    d_n = torch.tensor([n], dtype=torch.int32, device="cuda")
    scr = torch.full((A.scratch_bytes(n),), 0xAA, dtype=torch.uint8, device="cuda")
    seen = []
    for plan in (1 << 20, 1, 4096):
        A.set_tuning(plan_blocks=plan)
        out = torch.full((n * int(A.info.max_record_len),), 7, dtype=torch.uint8, device="cuda")
        offs = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        A.read_lookup(d_ids, out, offs, scr)
        A.sync_status()
        st = A.last_stats()
        got = out.cpu().numpy()
        assert got[:len(want_r)].tobytes() == want_r and (got[len(want_r):] == 7).all()
        out = torch.full((len(want_b) + 64,), 7, dtype=torch.uint8, device="cuda")
        A.decode_batch(d_reqs, d_n, n, out, offs, scr)
        A.sync_status()
        sb = A.last_stats()
        got = out.cpu().numpy()
        assert got[:len(want_b)].tobytes() == want_b and (got[len(want_b):] == 7).all()
        assert int(offs[-1]) == len(want_b)
        seen.append((st.closure_blocks, st.scratch_slots, st.covering, sb.closure_blocks, sb.scratch_slots, sb.covering))
    assert seen[0] == seen[1] == seen[2]
    A.set_tuning(plan_blocks=4096)


def test_one_block_means_never(arc):
    """plan_blocks 1 takes even a single read to the eight kernels (whose list
    head, control word 5, moves on; one workgroup leaves it at 0)."""
    x, starts, A = arc
    head = A.ws[A.ws.numel() - 512:].view(torch.int32)
    for plan, wide in ((4096, False), (1, True)):
        A.set_tuning(plan_blocks=plan)
        got, offs = A.read_lookup([3])
        A.sync_status()
        assert got[:int(offs[-1])].cpu().numpy().tobytes() == x[starts[3]:starts[4]]
        assert (int(head[5]) > 0) == wide
    A.set_tuning(plan_blocks=4096)
