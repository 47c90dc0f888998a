"""A watchdog limit of one poll does not fail valid archives: blocks that are
decoded by ticket wait for the blocks they copy from as long as it takes.
Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("beta", [0, 32])
def test_small_limit(beta):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, starts = fastq(n_records=12000, seed=3)
    arc = lz.Archive(lz.encode(x, kind=1, level_penalty=beta))
    assert arc.info.n_levels > 2
    arc.set_tuning(spin_limit=1)
    assert arc.tuning().spin_limit == 1
    out = torch.empty(len(x), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        out.fill_(7)
        arc.decode_all(out)
        arc.sync_status()
        assert out.cpu().numpy().tobytes() == x
        out.fill_(7)
        arc.decode_range(1, len(x) - 1, out=out)
        arc.sync_status()
        assert out[:-1].cpu().numpy().tobytes() == x[1:]
        ids = np.random.default_rng(1).integers(0, len(starts) - 1, 100)
        got, offs = arc.read_lookup(ids)
        arc.sync_status()
        want = b"".join(x[int(starts[r]):int(starts[r + 1])] for r in ids)
        assert got[:int(offs[-1])].cpu().numpy().tobytes() == want
