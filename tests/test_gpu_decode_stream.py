"""INT8 decode in launches that may read more than the memory-side cache holds: V rows come with the streaming hint, from
a copy of the tile loop of its own (from head_dim 128 on where rows are whole 128-byte lines).  The lengths are not known on the host here,
so the tables' width alone makes the launch count as large."""
import numpy as np
import pytest

from fs_inputs.workloads import INT8, ModelSpec, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("work_list", [0, 1])
@pytest.mark.parametrize("n_q", [8, 14])
@pytest.mark.parametrize("tokens,width", [(8, 18000), (27, 5400)])
def test_rows_with_the_streaming_hint(tokens, width, n_q, work_list):
    run(64, tokens, width, n_q, work_list)


@pytest.mark.parametrize("work_list", [0, 1])
@pytest.mark.parametrize("n_q", [8, 14])
@pytest.mark.parametrize("head_dim,tokens,width", [(128, 31, 2200), (128, 126, 560), (256, 31, 1100)])
def test_whole_lines_with_the_streaming_hint(head_dim, tokens, width, n_q, work_list):
    import oracle

    assert oracle.block_bytes(INT8, 2, head_dim, 1, tokens) // 2 % 128 == 0 and tokens * head_dim % 128 == 0  # a head's chunk, a head's K rows
    run(head_dim, tokens, width, n_q, work_list)


def run(head_dim, tokens, width, n_q, work_list):
    import gpu_harness
    import oracle
    import torch

    import paper_2509_06261_amd as fs

    lens = np.array([1, 7, 9, 31, 33, 65, 257, 2001], np.int32)
    assert len(lens) * width * tokens * 2 * 2 * (head_dim + 2) > 256 << 20  # sequences, table, KV heads, K and V, a token's row and scale
    slab = oracle.block_bytes(INT8, 2, head_dim, 1, tokens)
    par = gpu_harness.Parity(Workload("stream", slab, slab * 400, [ModelSpec("m", INT8, 2, head_dim, 1, n_q, lens, tag=68, tokens_per_block=tokens)], "shuffle"))
    try:
        gw = par.gw
        gw.pool_mem.fill_(0xFF)
        gw.set_option(fs.FS_OPT_DECODE_WORK_LIST, work_list)
        gw.populate([[0]])
        wide = torch.zeros((len(lens), width), dtype=torch.int32, device="cuda")
        wide[:, : gw.tables[0].shape[1]] = gw.tables[0]
        gw.tables[0] = wide
        batches, keep = gw.make_batches([0], host_lens=False)
        ws = gw.decode(batches)
        torch.cuda.synchronize()
        assert fs.fs_decode_status(ws) == 0
        print(par.check_model(0, [0], keep, with_bytes=False), fs.fs_pool_get_option(gw.pool, fs.FS_OPT_LAST_DECODE_KERNEL))
    finally:
        par.close()
