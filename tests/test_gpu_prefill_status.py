"""The status word of prefill launches without a preparation kernel, which one workgroup judges for the whole call: every share of
its threads that a sequence can get, entries at both ends of a table, and the ones that nobody reads."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, ModelSpec, Workload

pytestmark = pytest.mark.gpu


# (items of one tile each; from 256 on the launch is the one that may split items, below it is a small direct one)
@pytest.mark.parametrize("n_seq,length", [(1, 20000), (7, 3001), (65, 1100), (256, 1040), (300, 1100), (511, 1025)])
def test_entries_judged_by_one_workgroup(n_seq, length):
    import oracle
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    tokens = 16
    slab = oracle.block_bytes(FP16, 1, 128, 1, tokens)
    lens = np.full(n_seq, length, np.int32)
    gw = gpu_workload.GpuWorkload(Workload("status", slab, slab * 64, [ModelSpec("m", FP16, 1, 128, 1, 8, lens[:1] * 0 + 1, tag=5, tokens_per_block=tokens)],
                                           "identity"), zero_pool=True)
    try:
        need = -(-length // tokens)
        new = np.full(n_seq, 16, np.int32)
        idle = n_seq // 2 if n_seq > 2 else None  # a sequence that brings nothing: nobody reads its table
        if idle is not None:
            new[idle] = 0
        off = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
        off_d, lens_d = torch.from_numpy(off).cuda(), torch.from_numpy(lens).cuda()
        q = torch.randn((int(off[-1]), 8, 128), device="cuda", dtype=torch.float16)
        out = torch.empty_like(q)
        ws = torch.full((fs.fs_prefill_workspace_bytes(n_seq),), 0xFF, dtype=torch.uint8, device="cuda")
        table = torch.randint(0, 64, (n_seq, need + 3), dtype=torch.int32, device="cuda")

        def status():
            fs.fs_prefill_attention(gw.pool, gw.model_ids[0], 0, 8, 0.09, q, table, lens_d, off_d, off, out, None, ws)
            return fs.fs_decode_status(ws)

        table[:, need:] = -1
        if idle is not None:
            table[idle] = 64
        assert status() == 0
        for seq in sorted({0, n_seq - 1, n_seq // 3} - {idle}):
            for entry in (0, need - 1, need // 2):
                good = int(table[seq, entry])
                for bad in (64, -1):
                    table[seq, entry] = bad
                    assert status() == 4, (seq, entry, bad)
                table[seq, entry] = good
        lens_d[n_seq - 1] = (need + 3) * tokens + 1
        assert status() & 1
    finally:
        gw.close()
