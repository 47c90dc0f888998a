"""lz_open on workspace memory that already holds something: the closure's work
list must start empty.  An entry counts as pushed when its upper half equals
the call's epoch, so left-over words with a small upper half would be expanded
as blocks of the closure."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_open_clears_the_closure_list(orc):
    import paper_2606_18900_amd as lz
    from gen.fastq import fastq
    x, starts = fastq(n_records=4000, seed=5)
    arc = lz.Archive(orc.encode(x, kind=1, level_penalty=32))
    nb, L = arc.n_blocks, lz.lib()
    # every 64-bit word reads as "block 3, pushed in epoch 1"
    ws = torch.tensor([3, 1], dtype=torch.int32, device="cuda").repeat(arc.ws.numel() // 8 + 1)
    ws = ws.view(torch.uint8)[:arc.ws.numel()]
    h = C.c_void_p()
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.lz_open(C.c_void_p(arc.d_archive.data_ptr()), arc.d_archive.numel(), C.c_void_p(ws.data_ptr()),
                     ws.numel(), s, C.byref(h)) == 0
    try:
        # the list is the section before the control words (128 u32), 256-byte aligned
        at = ws.numel() - 512 - ((8 * nb + 255) & ~255)
        assert not np.any(ws[at:at + 8 * nb].cpu().numpy())
        # a call planned by the eight-kernel path
        tu = lz._lib.Tuning()
        assert L.lz_get_tuning(h, C.byref(tu)) == 0
        tu.plan_blocks = 1
        assert L.lz_set_tuning(h, C.byref(tu)) == 0
        ids = torch.arange(4000, device="cuda").flip(0)
        out = torch.zeros(4000 * int(arc.info.max_record_len), dtype=torch.uint8, device="cuda")
        offs = torch.empty(4001, dtype=torch.int64, device="cuda")
        scr = torch.empty(arc.scratch_bytes(4000), dtype=torch.uint8, device="cuda")
        p = lambda t: C.c_void_p(t.data_ptr())
        assert L.lz_read_lookup(h, p(ids), 4000, p(out), out.numel(), p(offs), p(scr), scr.numel(), s) == 0
        assert L.lz_sync_status(h, s) == 0
    finally:
        L.lz_close(h)
    want = b"".join(x[int(starts[r]):int(starts[r + 1])] for r in range(3999, -1, -1))
    assert int(offs[-1]) == len(want)
    assert out[:len(want)].cpu().numpy().tobytes() == want
