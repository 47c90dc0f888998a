"""Archives of few levels and many small blocks are decoded a level at a time,
all others by ticket (control word 2, the epoch, moves on): on both sides of
the line the bytes are the source's.  Exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bl,levels,by_ticket", [
    (6, 2, False), (6, 4, False), (6, 5, True), (10, 2, False), (10, 5, True), (11, 3, False), (11, 4, True),
    (12, 2, False), (12, 3, True), (13, 2, False), (13, 3, True), (14, 2, True)])
@pytest.mark.parametrize("wg", [1, 3])
def test_both_sides(bl, levels, by_ticket, wg):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    slots = wg * torch.cuda.get_device_properties(0).multi_processor_count
    x, starts = fastq(n_records=(2 * slots << bl) // 330 + 40, seed=4)
    a = lz.encode(x, kind=1, block_log2=bl, max_level=levels, level_penalty=0, hash_bits=22, segment_log2=22)
    arc = lz.Archive(a)
    assert arc.info.n_levels == levels and arc.n_blocks // 2 > slots
    arc.set_tuning(wg_per_cu=wg)
    epoch = arc.ws[arc.ws.numel() - 512:].view(torch.int32)[2:3]
    out = torch.full((len(x) + 16,), 7, dtype=torch.uint8, device="cuda")
    arc.decode_all(out)
    arc.sync_status()
    assert out[:len(x)].cpu().numpy().tobytes() == x and int(epoch) == int(by_ticket)
    # a range of half the file, and one too small to be decoded per level
    at = int(epoch)
    o, n = len(x) // 4 + 3, len(x) // 2
    out.fill_(7)
    arc.decode_range(o, n, out=out)
    arc.sync_status()
    assert out[:n].cpu().numpy().tobytes() == x[o:o + n] and int(epoch) == at + int(by_ticket)
    got, offs = arc.read_lookup(np.array([5]))
    arc.sync_status()
    assert got[:int(offs[-1])].cpu().numpy().tobytes() == x[int(starts[5]):int(starts[6])]
    assert int(epoch) == at + int(by_ticket) + 1


@pytest.mark.parametrize("bl,levels", [(8, 2), (8, 64), (10, 3), (12, 2)])
def test_split_streams(bl, levels):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, _ = fastq(n_records=25000 if bl == 12 else 9000, seed=4)
    A = lz.SplitArchive(lz.encode_split(x, block_log2=bl, max_level=levels, level_penalty=32 if levels == 64 else 0))
    out = torch.full((len(x) + 16,), 7, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        A.decode_all(out)
        A.sync_status()
        got = out.cpu().numpy()
        assert got[:len(x)].tobytes() == x and (got[len(x):] == 7).all()
        out.fill_(7)
