"""The verification hashes at the edges of their segments (64 bytes), chunks
(4096 bytes a wave) and rounds (8192 block hashes), against the source hashes
the encoder put into the directory and the oracle's tree hash.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SMALL = dict(min_match=16, hash_len=16, hash_bits=14, chain_depth=4)


@pytest.mark.parametrize("bl,n", [
    (14, 1), (14, 63), (14, 64), (14, 65), (14, 4095), (14, 4096), (14, 4097), (14, 12345),
    (14, 16383), (14, 16384), (14, 16385), (14, 5 * 16384 + 4096 + 33), (13, 8191), (13, 3 * 8192 + 1),
    (12, 4096), (12, 4097), (12, 40 * 4096 + 31), (11, 10 * 2048 + 5),
    (6, 64 * 511), (6, 64 * 8192), (6, 64 * 8193 + 7)])
def test_tree_and_block_hashes(orc, bl, n):
    import paper_2606_18900_amd as lz
    rng = np.random.default_rng(n + bl)
    x = rng.integers(0, 256, n, dtype=np.uint8).tobytes()
    a = orc.encode(x, block_log2=bl, **SMALL)
    arc = lz.Archive(a)
    out = arc.decode_all()
    tree = int(arc.verify(out).cpu().item()) & 0xFFFFFFFFFFFFFFFF
    arc.sync_status()                     # every block hash equals the directory's
    assert tree == orc.info(a).source_fnv
    bad = out.clone()
    bad[n // 2] ^= 1
    arc.verify(bad)
    with pytest.raises(lz.LzError) as e:
        arc.sync_status()
    assert e.value.code == -7             # LZ_ECORRUPT
    B = 1 << bl
    first = (n - 1) // B * B              # the last block alone
    arc.verify_range(out[first:].clone(), first, n - first)
    arc.sync_status()
