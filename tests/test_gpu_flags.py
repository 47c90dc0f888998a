"""Completion flags kept between launches: a block that nothing copies from
keeps its mark when it turns out corrupt, and the epochs' end is a launch like
any other."""
import struct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _flags(arc):
    """View of the workspace's flags: after the table (16 KiB), the queue and
    the 65 level offsets, each padded to 256 bytes."""
    nb = arc.n_blocks
    pad = lambda n: (n + 255) & ~255
    at = 16384 + pad(4 * nb) + pad(4 * 65)
    return arc.ws[at:at + 4 * nb].view(torch.int32)


def _archive(orc):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, _ = fastq(n_records=3000, seed=1)
    return lz, bytes(x), orc.encode(x, kind=1, level_penalty=32)


def test_corrupt_block_keeps_its_mark(orc):
    lz, x, a = _archive(orc)
    marks = _flags(lz.Archive(a)).cpu().numpy()
    leaf = int(np.nonzero(marks == -1)[0][-1])
    assert leaf and (marks == 0).any()
    d, pay = struct.unpack_from("<Q", a, 64)[0], struct.unpack_from("<Q", a, 88)[0]
    t = bytearray(a)
    t[pay + struct.unpack_from("<Q", a, d + 32 * leaf)[0]] = 9         # no such stream mode
    arc = lz.Archive(bytes(t))
    for _ in range(2):
        out = arc.decode_all()
        with pytest.raises(lz.LzError) as e:
            arc.sync_status()
        assert e.value.code == -7                                      # LZ_ECORRUPT
        assert _flags(arc).cpu().numpy()[leaf] == -1
        B = 1 << 14
        assert out[:B * leaf].cpu().numpy().tobytes() == x[:B * leaf]


def test_epochs_start_again(orc):
    lz, x, a = _archive(orc)
    arc = lz.Archive(a)
    ctl = arc.ws[arc.ws.numel() - 512:].view(torch.int32)
    ctl[2] = -4                                                        # the last decode's epoch: 2^32 - 4
    out = torch.empty(len(x), dtype=torch.uint8, device="cuda")
    for epoch in (-3, 0, 1, 2):
        out.fill_(7)
        arc.decode_all(out)
        arc.sync_status()
        assert out.cpu().numpy().tobytes() == x
        assert int(ctl[2]) == epoch
    # request calls: flags as long-gone launches left them, in both planners
    flags = _flags(arc)
    for plan in (4096, 1):
        arc.set_tuning(plan_blocks=plan)
        flags[flags != -1] = 1
        ctl[2] = -(1 << 28)
        for epoch in (1, 2):
            out.fill_(7)
            arc.decode_range(3, len(x) - 3, out=out)
            arc.sync_status()
            assert out[:-3].cpu().numpy().tobytes() == x[3:]
            assert int(ctl[2]) == epoch
