"""Decode where the tile code's loads and look-ups can go wrong: lengths around the ends of runs, tiles and blocks that are no
multiple of eight tokens, every format and head_dim of the MFMA kernel, both softmax layouts (up to four and more query heads
per KV head), launches with and without a work list -- over a pool whose unused bytes are all ones: keys, values, scales and
zero points past a sequence's end are NaN (an FP16 or FP8 element, a parameter) and must not reach its result."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, ModelSpec, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("work_list", [0, 1])
@pytest.mark.parametrize("head_dim,n_q", [(64, 8), (128, 8), (128, 14), (256, 8)])
@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("tokens", [8, 9, 27])
def test_rows_and_what_lies_behind_them(tokens, dtype, head_dim, n_q, work_list):
    import gpu_harness
    import oracle
    import paper_2509_06261_amd as fs

    slab = oracle.block_bytes(dtype, 2, head_dim, 1, tokens)
    lens = np.array([1, 7, 8, 9, 31, 32, 33, 63, 65, 100, 255, 257, 700, 2001], np.int32)
    spec = ModelSpec("m", dtype, 2, head_dim, 1, n_q, lens, tag=67, tokens_per_block=tokens)
    h = gpu_harness.Parity(Workload("rows", slab, slab * 600, [spec], "shuffle"))
    try:
        h.gw.pool_mem.fill_(0xFF)
        h.gw.set_option(fs.FS_OPT_DECODE_WORK_LIST, work_list)
        h.run_and_check([0], with_bytes=False)
        assert h.last_decode() == 2 or not work_list
    finally:
        h.close()
