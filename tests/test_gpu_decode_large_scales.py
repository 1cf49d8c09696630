"""INT4 decode where a softmax weight times a value's scale leaves the range of the half the matrix product takes it in: Inf in every
column whose stored code is not zero, even and odd ones alike, and no NaN."""
import numpy as np
import pytest

from fs_inputs.workloads import INT4, ModelSpec, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,n_q", [(64, 8), (128, 8), (128, 14), (256, 8)])
def test_an_infinite_weight_is_inf_in_odd_columns(head_dim, n_q):
    import oracle
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    n, at, tokens = 600, 100, 64
    slab = oracle.block_bytes(INT4, 2, head_dim, 1, tokens)
    wl = Workload("scales", slab, slab * 12, [ModelSpec("m", INT4, 2, head_dim, 1, n_q, np.array([n], np.int32), tag=9, src_f32=True, tokens_per_block=tokens)],
                  "identity")
    gw = gpu_workload.GpuWorkload(wl, zero_pool=True)
    try:
        gw.place()
        k = torch.zeros((n, 2, head_dim), dtype=torch.float32, device="cuda")
        v = torch.ones_like(k)
        k[at] = 0.5
        v[at, :, 0::2] = 7 * 12000.0  # codes 7 and 15 of a scale of 12000: 2^2.5 times that is above 65504
        v[at, :, 1::2] = 15 * 12000.0
        seq, pos = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")
        fs.fs_kv_append(gw.pool, gw.model_ids[0], 0, k, v, seq, pos, gw.tables[0])
        # 2.5 in the base-2 domain: below what moves the running reference (3), which the tiles before left at 0
        scale = 2.5 / np.log2(np.e) / (0.5 * head_dim)
        q = torch.ones((1, n_q, head_dim), dtype=torch.float16, device="cuda")
        out = torch.zeros_like(q)
        batch = fs.make_batch(gw.model_ids[0], 0, n_q, float(scale), q, gw.tables[0], gw.seq_lens[0], out, None, gw.lens[0])
        gw.decode([batch])
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.all(got[..., 0::2] == np.inf) and np.all(got[..., 1::2] == np.inf), got[0, 0, :4]
    finally:
        gw.close()
