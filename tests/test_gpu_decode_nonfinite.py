"""Decode over cached values that are not finite numbers (an fp32 key above 65504 is stored as Inf in an FP16 model; a
model that has gone NaN stores NaN): a NaN logit makes the outputs of the query heads that read it NaN wherever the token
stands -- in the share of any wave, in a sequence of one split or of several -- and changes no other output; a token whose
logit is -inf weighs nothing, also where a wave or a split holds no other token."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, KiB, ModelSpec, Workload

pytestmark = pytest.mark.gpu


class _Case:
    """Two sequences of one model with two KV heads, layer 0 filled; key rows can be overwritten in the pool."""

    def __init__(self, dtype, lens, split_bytes):
        import gpu_workload
        import paper_2509_06261_amd as fs

        self.fs, self.dtype, self.split_bytes = fs, dtype, split_bytes
        self.gw = gpu_workload.GpuWorkload(
            Workload("nf", 64 * KiB, 64 * 800 * KiB, [ModelSpec("m", dtype, 2, 128, 1, 8, np.array(lens, np.int32), tag=61, src_f32=dtype == INT4)],
                     "shuffle"), zero_pool=True, options={fs.FS_OPT_SPLIT_BYTES: split_bytes})
        self.gw.place()
        self.gw.populate([[0]])
        self.g = self.gw.geom[self.gw.model_ids[0]]

    def decode(self, q0=None, lens=None):
        import torch

        batches, keep = self.gw.make_batches([0], host_lens=lens is None)
        if q0 is not None:
            keep["q"][0][:, :, 0] = q0
        if lens is not None:
            ln = torch.tensor(lens, dtype=torch.int32, device=self.gw.device)
            batches[0].seq_lens = ln.data_ptr()
        ws = self.gw.decode(batches)
        torch.cuda.synchronize()
        assert self.fs.fs_decode_status(ws) == 0
        assert self.fs.fs_pool_get_option(self.gw.pool, self.fs.FS_OPT_LAST_DECODE_KERNEL) == (2 if self.split_bytes else 4)
        return keep["out"][0].cpu().numpy(), keep["lse"][0].cpu().numpy()

    def key_bytes(self, seq, token, head, new=None):
        """The first two bytes of a key (FP16), its first byte (FP8) or its scale (INT8, INT4); replaced if ``new`` is given."""
        g, T = self.g, self.g.tokens_per_block
        at = int(self.gw.tables_host[0][seq, token // T]) * g.block_budget + head * g.head_chunk
        if self.dtype in (FP16, FP8):
            at += (token % T) * g.row_bytes
        else:
            at += 2 * g.kv_tile + (token % T) * g.param_bytes
        part = self.gw.pool_mem[at: at + (1 if self.dtype == FP8 else 2)]
        old = part.cpu().numpy().copy()
        if new is not None:
            import torch
            part.copy_(torch.from_numpy(np.asarray(new, np.uint8)))
        return old


@pytest.mark.parametrize("split_bytes", [0, 16 * KiB])
@pytest.mark.parametrize("lens,tokens", [([140, 90], [0, 33, 64, 97, 139]), ([5000, 90], [3, 2499, 4970, 4999])])
@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
def test_nan_logit(dtype, lens, tokens, split_bytes):
    c = _Case(dtype, lens, split_bytes)
    try:
        out0, lse0 = c.decode()
        assert np.isfinite(out0).all() and np.isfinite(lse0).all()
        nan = [0x7F] if dtype == FP8 else [0x00, 0x7E]
        for token in tokens:
            for head in range(2):
                old = c.key_bytes(0, token, head, nan)
                out, lse = c.decode()
                c.key_bytes(0, token, head, old)
                hit = np.zeros((2, 8), bool)
                hit[0, 4 * head: 4 * head + 4] = True
                assert np.isnan(out[hit]).all() and np.isnan(lse[hit]).all(), (token, head)
                assert np.array_equal(out[~hit], out0[~hit]) and np.array_equal(lse[~hit], lse0[~hit]), (token, head)
    finally:
        c.gw.close()


@pytest.mark.parametrize("split_bytes", [0, 16 * KiB])
@pytest.mark.parametrize("n,cut", [(97, 96), (40, 32), (161, 128), (2689, 2688)])
def test_minus_infinity_logits(n, cut, split_bytes):
    """The tokens from ``cut`` on have a logit of -inf: the result is that of the sequence cut there."""
    c = _Case(FP16, [n, 50], split_bytes)
    try:
        for t in range(cut, n):
            for head in range(2):
                c.key_bytes(0, t, head, [0x00, 0xFC])  # -inf, times a positive query element
        out, lse = c.decode(q0=1.0)
        out0, lse0 = c.decode(q0=1.0, lens=[cut, 50])
        # the same weights, summed in another order, in an fp16 result of magnitude <= 2
        assert np.abs(out.astype(np.float64) - out0).max() <= 2e-3 and np.abs(lse - lse0).max() <= 1e-4
    finally:
        c.gw.close()
