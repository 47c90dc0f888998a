"""Matches that repeat themselves, of every period around the 16-byte pieces
and of lengths around the pieces, the wave and the block, beginning inside the
block or in the one before, against the plain bytes.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 61, 64, 100, 255, 256, 500, 513, 2000])
def test_period(d):
    import paper_2606_18900_amd as lz
    rng = np.random.default_rng(d)
    parts = []
    for n in (16, 17, 40, 63, 64, 65, 127, 129, 255, 256, 257, 300, 1000, 1024, 1025, 5000, 16384, 33000, 70000):
        head = rng.integers(0, 256, int(rng.integers(20, 90)), dtype=np.uint8).tobytes()
        unit = rng.integers(0, 256, d, dtype=np.uint8).tobytes()
        parts.append(head + (unit * (n // d + 2))[:n + d])
    x = b"".join(parts)
    for penalty in (0, 32):
        arc = lz.Archive(lz.encode(x, level_penalty=penalty, hash_bits=16))
        for mode in (0, 1):
            arc.set_tuning(sync_mode=mode)
            out = arc.decode_all()
            arc.sync_status()
            assert out.cpu().numpy().tobytes() == x, (penalty, mode)
        o = len(x) - 60000
        got = arc.decode_range(o, 30011)
        arc.sync_status()
        assert got.cpu().numpy().tobytes() == x[o:o + 30011]
