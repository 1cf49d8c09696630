"""GPU parity of decode launches without a work list (one workgroup per sequence, split and KV head) at their edges,
against the CPU oracle: lengths around the tiles and the four waves' shares, one split and several, several formats in
one launch, odd tokens per block, and the status word, which no kernel clears before the launch.  Tolerances are the
harness's."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, KiB, MiB, ModelSpec, Workload

pytestmark = pytest.mark.gpu


def _check(wl, layers):
    import gpu_harness

    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        print(par.gw.T, par.run_and_check(layers))
        assert par.last_decode() == 4  # (the kernel this file is about)
    finally:
        par.close()


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,kv_heads,group", [(64, 4, 1), (64, 2, 8), (128, 2, 4), (128, 3, 16), (256, 2, 3), (256, 2, 16)])
def test_short_sequences(dtype, head_dim, kv_heads, group):
    lens = np.array([1, 7, 8, 9, 31, 32, 33, 127, 128, 129, 257, 400], np.int32)
    _check(Workload("dd", 160 * KiB, 160 * 400 * KiB,
                    [ModelSpec("m", dtype, kv_heads, head_dim, 2, kv_heads * group, lens, tag=51, src_f32=dtype == INT4)], "shuffle"), [1])


@pytest.mark.parametrize("dtype,head_dim,lens", [(FP16, 128, [9000, 1, 2500, 4096]), (INT4, 128, [12000, 333]), (FP8, 64, [16000]),
                                                 (INT8, 256, [5000, 4999, 17])])
def test_sequences_in_several_splits(dtype, head_dim, lens):
    lens = np.array(lens, np.int32)
    _check(Workload("ds", 96 * KiB, 96 * 2000 * KiB, [ModelSpec("m", dtype, 2, head_dim, 2, 8, lens, tag=52, src_f32=dtype == INT4)],
                    "shuffle"), [0])


def test_several_formats_in_one_launch():
    la, lb, lc = (np.array(x, np.int32) for x in ([3000, 5, 700, 64], [90] * 20 + [2000], [1, 4000]))
    _check(Workload("dm", 96 * KiB, 96 * 1500 * KiB,
                    [ModelSpec("a", FP16, 4, 128, 1, 16, la, tag=53), ModelSpec("b", INT4, 2, 128, 2, 2, lb, tag=54, src_f32=True),
                     ModelSpec("c", FP8, 1, 128, 1, 8, lc, tag=55)], "interleave"), [0, 1, 0])


@pytest.mark.parametrize("n", [40, 6000])  # one split; several
def test_status_without_preparation(n):
    """Whatever the workspace held, the status is this call's alone: 0, bit 0 for a length out of range, bit 2 for an entry
    outside the pool inside a length -- and an entry past a sequence's end is neither read nor reported."""
    import torch

    import paper_2509_06261_amd as fs

    slab, n_slabs = 64 * KiB, 1024
    mem = torch.zeros(slab * n_slabs, dtype=torch.uint8, device="cuda")
    pool = fs.fs_pool_create(slab, mem.numel(), mem)
    try:
        _, model = fs.fs_model_register(pool, fs.FS_KV_FP16, 2, 128, 1)
        T = fs.fs_model_geometry(pool, model).tokens_per_block
        nb = -(-n // T)
        table = np.full((3, nb + 1), 1 << 20, np.int32)
        table[:, :nb] = fs.fs_blocks_alloc(pool, model, 3 * nb)[1].reshape(3, nb)
        q = torch.ones((3, 8, 128), dtype=torch.float16, device="cuda")

        def status(lens, table):
            t, ln, out = torch.from_numpy(table).cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda"), torch.empty_like(q)
            b = [fs.make_batch(model, 0, 8, 0.1, q, t, ln, out, None, None)]
            ws = torch.full((fs.fs_decode_workspace_bytes(pool, b),), 0xff, dtype=torch.uint8, device="cuda")
            fs.fs_decode_attention_multi(pool, b, ws)
            torch.cuda.synchronize()
            assert fs.fs_pool_get_option(pool, fs.FS_OPT_LAST_DECODE_KERNEL) == 4
            assert bool((out == 0).all())  # zero values in the pool, whatever block stands in for a bad entry
            return fs.fs_decode_status(ws)

        assert status([n, 1, n // 2], table) == 0
        assert status([n, 0, n // 2], table) == 1
        bad = table.copy()
        bad[2, 0] = -1
        assert status([n, 1, n // 2], bad) == 4
        assert status([n + 2 * T, 1, 3], bad) == 5  # (clamped to the table's last block)
    finally:
        fs.fs_pool_destroy(pool)


@pytest.mark.parametrize("dtype,head_dim,group", [(FP16, 128, 4), (INT4, 128, 1), (FP8, 64, 8), (INT8, 256, 4), (FP16, 256, 3)])
def test_sequences_longer_on_the_device_than_on_the_host(dtype, head_dim, group):
    """seq_lens_host only sizes the launch (a captured step replayed while its sequences grow): the last split of a
    sequence takes whatever it holds beyond the host's length, here up to dozens of the address table's segments."""
    import torch

    import gpu_harness

    lens = np.array([6000, 20, 9001, 700, 1], np.int32)
    known = np.array([600, 20, 333, 700, 650], np.int32)
    par = gpu_harness.Parity(Workload("dl", 96 * KiB, 96 * 700 * KiB,
                                      [ModelSpec("m", dtype, 2, head_dim, 1, 2 * group, lens, tag=56, src_f32=dtype == INT4)],
                                      "shuffle"), zero_pool=True)
    try:
        par.gw.populate([[0]])
        batches, keep = par.gw.make_batches([0])
        batches[0].seq_lens_host = known.ctypes.data
        ws = par.gw.decode(batches)
        torch.cuda.synchronize()
        assert par.fs.fs_decode_status(ws) == 0 and par.last_decode() == 4
        print(par.check_model(0, [0], keep))
    finally:
        par.close()
