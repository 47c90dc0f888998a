"""Blocks decoded by ticket in one launch (sync_mode 0) against the plain
bytes and against one launch per level (sync_mode 1): outputs that share cache
lines between blocks (not aligned to 128 bytes), blocks smaller than a line,
blocks that copy from more than 256 others, buffers reused by other calls.
Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lz():
    import paper_2606_18900_amd as lz
    return lz


def _decode(arc, x, buf, shift, mode):
    arc.set_tuning(sync_mode=mode, req_sync_mode=mode)
    buf.fill_(7)
    arc.decode_all(out=buf[shift:shift + len(x)])
    arc.sync_status()
    got = buf.cpu().numpy()
    assert got[shift:shift + len(x)].tobytes() == x
    assert (got[:shift] == 7).all() and (got[shift + len(x):] == 7).all()


@pytest.mark.parametrize("bl,recs,beta", [(14, 3000, 32), (14, 3000, 0), (10, 1500, 4), (7, 300, 1), (6, 200, 1)])
def test_alignment_and_reuse(orc, lz, bl, recs, beta):
    from gen.fastq import fastq
    p = dict(kind=1, block_log2=bl, level_penalty=beta)
    x, _ = fastq(n_records=recs, seed=11)
    y, _ = fastq(n_records=recs, seed=12)
    A, B = lz.Archive(orc.encode(x, **p)), lz.Archive(orc.encode(y, **p))
    assert A.info.n_levels > 2
    buf = torch.empty(max(len(x), len(y)) + 512, dtype=torch.uint8, device="cuda")
    for shift in (0, 16, 48, 64, 128):
        for mode in (0, 1, 0):
            _decode(A, x, buf, shift, mode)
            _decode(B, y, buf, shift, mode)
    A.set_tuning(req_sync_mode=0)
    Bs = 1 << bl
    for o in (0, 16, 112, 128, Bs + 32, Bs - 16):
        for shift in (0, 16, 128):
            n = len(x) - o - 5
            buf.fill_(7)
            A.decode_range(o, n, out=buf[shift:shift + n])
            A.sync_status()
            assert buf[shift:shift + n].cpu().numpy().tobytes() == x[o:o + n], (o, shift)


def test_many_dependencies(lz):
    # two blocks of 48-byte pieces of 330 earlier blocks of noise, in another order
    rng = np.random.default_rng(5)
    B, nb = 1 << 14, 330
    head = rng.integers(0, 256, nb * B, dtype=np.uint8)
    tail = b"".join(head[b * B + int(o):b * B + int(o) + 48].tobytes()
                    for r in range(2) for b, o in zip(rng.permutation(nb), rng.integers(0, B - 48, nb)))
    x = head.tobytes() + tail
    arc = lz.Archive(lz.encode(x, hash_bits=22, level_penalty=0))
    ptr = int.from_bytes(arc.d_archive[72:80].cpu().numpy().tobytes(), "little")
    deps = arc.d_archive[ptr:ptr + 8 * (arc.n_blocks + 1)].clone().view(torch.int64).cpu().numpy()
    assert np.diff(deps).max() > 256
    buf = torch.empty(len(x) + 256, dtype=torch.uint8, device="cuda")
    for shift in (0, 16):
        for mode in (0, 1, 0):
            _decode(arc, x, buf, shift, mode)
    out = arc.decode_range(len(x) - 9000, 9000)
    arc.sync_status()
    assert out.cpu().numpy().tobytes() == x[-9000:]
