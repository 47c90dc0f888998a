"""Literals that are stored, or all one byte, at the edges of their 16-byte
pieces: alone in their block and cut into short runs between matches, against
the plain bytes.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _check(lz, x, block):
    arc = lz.Archive(lz.encode(x, block_log2=block, hash_bits=16))
    for mode in (0, 1):
        arc.set_tuning(sync_mode=mode)
        out = arc.decode_all()
        arc.sync_status()
        assert out.cpu().numpy().tobytes() == x, mode
    o = len(x) // 3
    got = arc.decode_range(o, len(x) - o)
    arc.sync_status()
    assert got.cpu().numpy().tobytes() == x[o:]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 4095, 4096, 4097, 4111, 16383, 16400, 16384 * 3 + 5])
@pytest.mark.parametrize("block", [12, 14])
def test_stored(n, block):
    import paper_2606_18900_amd as lz
    x = np.random.default_rng(n).integers(0, 256, n, dtype=np.uint8).tobytes()
    _check(lz, x, block)
    _check(lz, bytes([65]) * min(n, 31), block)


@pytest.mark.parametrize("run", [1, 3, 15, 16, 17, 40, 200])
@pytest.mark.parametrize("few", [False, True])
def test_runs(run, few):
    """Runs of `run` new bytes between copies of 40: of a byte that may take any
    value (stored) or of one value only (one symbol)."""
    import paper_2606_18900_amd as lz
    rng = np.random.default_rng(run)
    head = rng.integers(0, 256, 3000, dtype=np.uint8).tobytes()
    parts = [head]
    for k in range(400):
        o = int(rng.integers(0, 2900))
        parts.append(bytes([7]) * run if few else rng.integers(0, 256, run, dtype=np.uint8).tobytes())
        parts.append(head[o:o + 40])
    _check(lz, b"".join(parts), 14)
