"""Records of a split container put back together 16 bytes at a time: lines
shorter than a piece, around one and two pieces, long ones, ranges that cut
records, and the four streams decoded in one launch or one after the other.
Exact, nothing written outside."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _text(lengths, seed):
    rng = np.random.default_rng(seed)
    out, starts = bytearray(), [0]
    for k, n in enumerate(lengths):
        out += b"@" + b"r" * int(rng.integers(0, 40)) + b"%d\n" % k
        out += rng.choice(np.frombuffer(b"ACGT", np.uint8), n).tobytes() + b"\n+\n"
        out += rng.integers(35, 70, n, dtype=np.uint8).tobytes() + b"\n"
        starts.append(len(out))
    return bytes(out), starts


@pytest.mark.parametrize("lengths,bl", [
    ([1], 14), (list(range(1, 70)) * 4, 14), (list(range(1, 70)) * 4, 8),
    ([150] * 900, 14), ([5000, 3, 17, 40000, 16, 15] * 5, 14)])
def test_lines(lengths, bl):
    import paper_2606_18900_amd as lz
    x, starts = _text(lengths, len(lengths))
    A = lz.SplitArchive(lz.encode_split(x, block_log2=bl, hash_bits=16))
    for mode in (0, 1, 0):
        A.set_tuning(sync_mode=mode)
        for shift in (0, 1, 13):
            buf = torch.full((len(x) + 64,), 7, dtype=torch.uint8, device="cuda")
            A.ws[:256].fill_(0)
            A.decode_all(buf[shift:shift + len(x)])
            A.sync_status()
            got = buf.cpu().numpy()
            assert got[shift:shift + len(x)].tobytes() == x, (mode, shift)
            assert (got[:shift] == 7).all() and (got[shift + len(x):] == 7).all()
    rng = np.random.default_rng(1)
    for _ in range(12):
        o = int(rng.integers(0, len(x)))
        n = int(min(len(x) - o, np.exp(rng.random() * np.log(len(x)))) or 1)
        buf = torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda")
        A.decode_range(o, n, out=buf[1:1 + n])
        A.sync_status()
        got = buf.cpu().numpy()
        assert got[1:1 + n].tobytes() == x[o:o + n] and got[0] == 7 and (got[1 + n:] == 7).all()
    ids = rng.integers(0, len(lengths), 50)
    out, offs = A.read_lookup(ids)
    A.sync_status()
    o = offs.cpu().numpy()
    want = [x[starts[i]:starts[i + 1]] for i in ids]
    assert out.cpu().numpy()[:o[-1]].tobytes() == b"".join(want)
    assert np.diff(o).tolist() == [len(w) for w in want]
