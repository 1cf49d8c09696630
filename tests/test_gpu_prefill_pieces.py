"""Prefill launches that certainly leave pieces of items in the workspace (every test here looks for them there): items of
several tiles whose diagonals are cut, sequences dealt tile by tile, pieces that begin in a later segment of the address
table, one to forty KV heads, repeats over a workspace that held anything, and a replayed capture."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, ModelSpec, Workload

pytestmark = pytest.mark.gpu

GROUPS, PIECE_BYTES = 256, 133120
PIECES_BYTES = 8 * GROUPS + 2 * GROUPS * PIECE_BYTES  # counters, then two places a workgroup

# KV heads, query heads per KV head, tokens per block, contexts, new tokens, sequences checked against the oracle
SHAPES = {
    # five chunks of eight tiles each, dealt one tile of each sequence in turn
    "even": (8, 4, 16, [1500, 2600, 3301, 4000, 6000], [512] * 5, [0]),
    # one tile each; a segment of the table holds 4480 tokens, so pieces begin in the second and third and at odd slots
    "segments": (8, 4, 9, [9100, 8200, 7000] + [1500] * 31, [33] * 34, [0, 33]),
    # unequal numbers of tiles, the last one ragged; three query heads (tiles of 80 tokens)
    "diagonals": (8, 4, 32, [6100, 5200, 900, 1300, 2500], [700, 512, 900, 130, 300], [2, 3]),
    "three-heads": (8, 3, 13, [6100, 5200, 900, 1300, 2500], [700, 512, 900, 430, 300], [2]),
    "one-kv-head": (1, 8, 21, [700, 1000, 1500, 2300, 3000, 3500, 4100, 6000], [520, 1000, 1024, 1000, 1100, 1024, 1400, 1024], [0, 2]),
    "two-kv-heads": (2, 4, 24, [900, 1100, 1500, 2300, 3000, 3500, 4100, 6000], [900, 1000, 1024, 1000, 1100, 1024, 1024, 1024], [0, 2]),
    "four-kv-heads": (4, 4, 12, [900, 1100, 1500, 2300, 3000, 3500, 4100, 6000], [500, 512, 512, 600, 512, 512, 500, 512], [0, 3]),
    "five-kv-heads": (5, 2, 16, [1100, 1500, 2300, 3000, 3500, 4100, 6000], [1000, 1024, 1000, 1100, 1024, 1300, 1324], [0]),
    # last tiles of 26 and 36 tokens (four and five waves of eight with tokens, whose steps weigh less), cut like the whole ones
    "light": (8, 4, 16, [9000, 8100] + [1500] * 10, [154, 164] + [154] * 10, [0, 1]),
    "multi-head": (40, 1, 15, [400, 900, 1500, 5000], [300, 256, 600, 700], [0, 1]),
}


def workload(dtype, shape):
    import oracle

    kv_heads, group, tokens, lens, new, seqs = SHAPES[shape]
    slab = oracle.block_bytes(dtype, kv_heads, 128, 1, tokens)
    blocks = sum(-(-n // tokens) for n in lens) + 50
    spec = ModelSpec("m", dtype, kv_heads, 128, 1, kv_heads * group, np.array(lens, np.int32), tag=71, src_f32=dtype == INT4,
                     tokens_per_block=tokens)
    return Workload("pieces", slab, slab * blocks, [spec], "shuffle"), np.array(new, np.int32), seqs


def pieces_left(ws, n_seq):
    """Which of the pieces' places a launch wrote, in a workspace that was all 0xff; its counters read zero again."""
    import torch

    import paper_2509_06261_amd as fs

    base = fs.fs_prefill_workspace_bytes(n_seq) - PIECES_BYTES
    counters = ws[base : base + 8 * GROUPS].view(torch.int64).cpu().numpy()
    used = (ws[base + 8 * GROUPS : base + PIECES_BYTES].view(2 * GROUPS, PIECE_BYTES) != 0xFF).any(dim=1).cpu().numpy()
    first = used[1::2]  # (an item's first piece lies in its workgroup's second place)
    assert np.all(counters == np.where(first, 0, -1))
    assert first.sum() > 0 and used.sum() >= 2 * first.sum()
    return int(first.sum()), int(used.sum())


class Watched:
    """The binding with every prefill workspace filled with ones first, and kept."""

    def __init__(self, fs):
        self.fs, self.ws = fs, None

    def __getattr__(self, name):
        return getattr(self.fs, name)

    def fs_prefill_attention(self, *args):
        self.ws = args[-1]
        self.ws.fill_(0xFF)
        return self.fs.fs_prefill_attention(*args)


@pytest.mark.parametrize("shape,dtype", [("even", FP8), ("even", INT4), ("segments", FP16), ("segments", INT8), ("diagonals", FP16),
                                         ("diagonals", INT4), ("three-heads", INT8), ("one-kv-head", FP8), ("two-kv-heads", INT4),
                                         ("four-kv-heads", FP16), ("five-kv-heads", INT8), ("multi-head", INT4), ("light", FP16), ("light", INT8)])
def test_pieces_against_the_oracle(shape, dtype):
    import gpu_harness

    wl, new, seqs = workload(dtype, shape)
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[0]])
        par.fs = Watched(par.fs)
        print(par.prefill_and_check(0, 0, new, seqs))
        items, pieces = pieces_left(par.fs.ws, len(new))
        print(f"{shape}: {items} items in {pieces} pieces")
        if shape == "segments":
            assert pieces > 2 * items  # (items in more than two pieces)
    finally:
        par.close()


@pytest.mark.parametrize("shape,dtype", [("even", INT4), ("segments", FP16), ("diagonals", FP8), ("diagonals", INT8)])
def test_the_same_bits_whoever_adds_them_up(shape, dtype):
    """Repeats of a launch with pieces, eager and as a replayed capture, over a workspace of ones, of noise, of zeros and as
    the launch before left it; the rows that whole items give in a
    workspace without room differ by roundings only."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    wl, new, _ = workload(dtype, shape)
    gw = gpu_workload.GpuWorkload(wl, zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        n, n_q = len(new), wl.models[0].n_q_heads
        off = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
        off_d = torch.from_numpy(off).cuda()
        q = torch.randn((int(off[-1]), n_q, 128), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda", dtype=torch.float16)
        out, lse = torch.empty_like(q), torch.empty(q.shape[:2], device="cuda")
        full = fs.fs_prefill_workspace_bytes(n)
        ws = torch.full((full,), 0xFF, dtype=torch.uint8, device="cuda")

        def run(ws):
            fs.fs_prefill_attention(gw.pool, gw.model_ids[0], 0, n_q, 0.09, q, gw.tables[0], gw.seq_lens[0], off_d, off, out, lse, ws)

        run(ws)
        assert fs.fs_decode_status(ws) == 0
        items, pieces = pieces_left(ws, n)
        first = out.clone(), lse.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(ws)
        for k in range(24):
            out.fill_(float("nan"))
            lse.fill_(float("nan"))
            if k % 6 == 2:
                ws.random_(0, 256)
            elif k % 6 == 4:
                ws.zero_()
            elif k % 6 == 5:
                ws.fill_(0xFF)
            graph.replay() if k % 2 else run(ws)
            torch.cuda.synchronize()
            assert torch.equal(out, first[0]) and torch.equal(lse, first[1]), k
            if k % 6 == 5:
                assert pieces_left(ws, n) == (items, pieces)
        small = ws[: full - PIECES_BYTES]
        before = ws.clone()
        run(small)
        assert fs.fs_decode_status(small) == 0
        assert torch.equal(ws[full - PIECES_BYTES :], before[full - PIECES_BYTES :])  # (no piece was left)
        # one rounding of the fp16 result each (2^-11 of it), the weights' roundings against another reference beside it
        assert bool(((out.float() - first[0].float()).abs() <= first[0].float().abs() * 2.0 ** -10 + 1e-3).all())
        assert float((lse - first[1]).abs().max()) <= 1e-3
    finally:
        gw.close()
