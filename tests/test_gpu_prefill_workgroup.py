"""GPU parity of the workgroup prefill kernel at its edges, against the CPU oracle row by row: head_dims beside 128, prompt
lengths around the 32-token sub-tiles, 128-token steps and 64- to 256-token items, waves whose queries end early in a
step, chunks shorter than a wave's share.  Tolerances are the harness's (derived there from the fp16 roundings)."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, KiB, MiB, ModelSpec, Workload

pytestmark = pytest.mark.gpu

EDGES = np.array([1, 31, 32, 33, 64, 65, 127, 128, 129, 255, 257, 300, 511], np.int32)
CHUNKS = np.array([1, 0, 32, 1, 17, 64, 16, 128, 33, 200, 1, 300, 65], np.int32)


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,group", [(64, 4), (64, 1), (64, 3), (128, 4), (128, 1)])
def test_workgroup_kernel_edges(dtype, head_dim, group, monkeypatch):
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    wl = Workload("pfwg", 96 * KiB, 96 * 400 * KiB,
                  [ModelSpec("m", dtype, 2, head_dim, 2, 2 * group, EDGES, tag=41, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[1]])
        print("T", par.gw.T, par.prefill_and_check(0, 1, EDGES), par.prefill_and_check(0, 1, CHUNKS))
        ran = fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL)
        assert ran & 0xffff == (16 | 8 << 8), ran
        assert bool(ran >> 16 & 1) == (head_dim == 128 and dtype in (INT8, INT4))  # exact codes at head_dim 64
    finally:
        par.close()
