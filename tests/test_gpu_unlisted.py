"""Archives whose dependency lists leave out a block that another copies from
(every check of the lists against each other still passes): blocks of lower
levels are there when a level is decoded, listed or not, so whole-file decodes
and ranges that cover both blocks give the source.  Exact."""
import struct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

B = 1 << 14


def _three_blocks(lz):
    """Stored block 0, block 1 of coded literals (the slower one), block 2 of
    pieces of both; then block 1 is taken off block 2's list."""
    rng = np.random.default_rng(8)
    a = rng.integers(0, 256, B, dtype=np.uint8).tobytes()
    b = rng.choice(np.frombuffer(b"ACGT", np.uint8), B).tobytes()
    c = b"".join(s[o:o + 64] for k in range(B // 128) for s, o in ((a, 128 * k), (b, 128 * (B // 128 - 1 - k))))
    x = a + b + c
    t = bytearray(lz.encode(x, level_penalty=0, hash_bits=16))
    ptr, idx = struct.unpack_from("<QQ", t, 72)
    assert struct.unpack_from("<4Q", t, ptr) == (0, 0, 0, 2) and struct.unpack_from("<2I", t, idx) == (0, 1)
    struct.pack_into("<Q", t, ptr + 24, 1)
    return x, bytes(t)


def _swapped(orc):
    from gen.fastq import fastq
    from tests.ref.tamper import swap_dependency
    x, _ = fastq(n_records=3000, seed=1)
    return bytes(x), swap_dependency(orc.encode(x, kind=1, level_penalty=32))[0]


@pytest.mark.parametrize("which", ["three", "swapped"])
def test_sources_that_are_not_listed(orc, which):
    import paper_2606_18900_amd as lz
    x, t = _three_blocks(lz) if which == "three" else _swapped(orc)
    arc = lz.Archive(t)
    scratch = torch.empty(arc.scratch_bytes(1), dtype=torch.uint8, device="cuda")
    out = torch.empty(len(x), dtype=torch.uint8, device="cuda")
    for plan in (4096, 1):
        arc.set_tuning(plan_blocks=plan)
        for _ in range(4):
            out.fill_(7)
            arc.decode_all(out)
            arc.sync_status()
            assert out.cpu().numpy().tobytes() == x
            out.fill_(7)
            scratch.fill_(0xAA)
            arc.decode_range(0, len(x), out=out, scratch=scratch)
            arc.sync_status()
            assert out.cpu().numpy().tobytes() == x


def test_complete_lists_stay_in_one_launch(orc):
    """What the encoder writes is decoded by ticket: the epoch of the last such
    launch advances (control word 2)."""
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, _ = fastq(n_records=3000, seed=1)
    arc = lz.Archive(orc.encode(x, kind=1, level_penalty=32))
    arc.decode_all()
    arc.sync_status()
    assert int(arc.ws[arc.ws.numel() - 512:].view(torch.int32)[2]) == 1
