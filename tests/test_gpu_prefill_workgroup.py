"""GPU parity of the workgroup prefill kernel at its edges, against the CPU oracle row by row: head_dims beside 128, prompt
lengths around the 32-token sub-tiles, 128-token steps and 64- to 256-token items, waves whose queries end early in a
step, chunks shorter than a wave's share.  Tolerances are the harness's (derived there from the fp16 roundings)."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, FP8, INT4, INT8, KiB, MiB, ModelSpec, Workload

pytestmark = pytest.mark.gpu

EDGES = np.array([1, 31, 32, 33, 64, 65, 127, 128, 129, 255, 257, 300, 511], np.int32)
CHUNKS = np.array([1, 0, 32, 1, 17, 64, 16, 128, 33, 200, 1, 300, 65], np.int32)
CHUNKS_256 = np.array([1, 0, 32, 1, 32, 64, 63, 128, 64, 200, 1, 300, 255], np.int32)  # half to one item per compute unit


# (head_dim 64 and 256 take the kernel by the size of the launch alone: as many KV heads as that needs)
@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,kv_heads,group", [(64, 13, 4), (64, 20, 1), (64, 15, 3), (128, 2, 4), (128, 2, 1), (256, 2, 4), (256, 2, 3)])
def test_workgroup_kernel_edges(dtype, head_dim, kv_heads, group, monkeypatch):
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    wl = Workload("pfwg", 96 * KiB, 96 * 400 * KiB,
                  [ModelSpec("m", dtype, kv_heads, head_dim, 2, kv_heads * group, EDGES, tag=41, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[1]])
        for n_new in (EDGES, CHUNKS_256 if head_dim == 256 else CHUNKS):
            print("T", par.gw.T, par.prefill_and_check(0, 1, n_new))
            ran = fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL)
            assert ran & 0xffff == (4 | 4 << 8 if head_dim == 256 else 16 | 8 << 8), ran
            assert bool(ran >> 16 & 1) == (head_dim == 128 and dtype in (INT8, INT4))  # exact codes at head_dim 64
    finally:
        par.close()


@pytest.mark.parametrize("head_dim,dtype,kernel", [(64, FP16, 1), (256, FP8, 1), (128, FP16, 16 | 8 << 8)])
def test_column_blocks_option_concerns_head_dim_128(head_dim, dtype, kernel, monkeypatch):
    """A pool-wide FS_OPT_PREFILL_COLUMN_BLOCKS of 16 leaves the models of other head_dims on the kernel that the size of
    their launch asks for: here a few items, and at head_dim 256 FP8 prompts of more items than compute units."""
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    lens = EDGES if head_dim == 256 else np.array([3, 40], np.int32)
    wl = Workload("pfcb", 256 * KiB, 256 * 200 * KiB, [ModelSpec("m", dtype, 4, head_dim, 2, 16, lens, tag=44)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[1]])
        par.prefill_and_check(0, 1, lens)
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == kernel
    finally:
        par.close()


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8])
def test_four_wave_option_leaves_launches_below_an_item_per_unit_alone(dtype, monkeypatch):
    """Between the direct launches and those with a 16-block item per compute unit: sums over the unrounded weights and
    exact codes, which the 4-wave kernels of FS_OPT_PREFILL_WAVES = 4 do not have."""
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_WAVES: 4})
    wl = Workload("pfnw", 384 * KiB, 384 * 200 * KiB, [ModelSpec("m", dtype, 5, 128, 2, 20, EDGES, tag=45)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[1]])
        par.prefill_and_check(0, 1, EDGES)
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (16 | 8 << 8)
    finally:
        par.close()


@pytest.mark.parametrize("head_dim,kv_heads,group,kernel", [(64, 16, 4, 16 | 8 << 8), (64, 6, 4, 8 | 8 << 8), (128, 3, 4, 8 | 8 << 8),
                                                            (128, 5, 1, 8 | 8 << 8), (128, 12, 4, 16 | 8 << 8), (256, 4, 4, 4 | 4 << 8)])
def test_infinite_value_reaches_no_row_before_its_block(head_dim, kv_heads, group, kernel):
    """An Inf among the values (an fp32 value above 65504 in an FP16 model) at token t: the rows of earlier blocks of 16
    columns are what they are without it, and the rows from t on are not finite."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    lens = np.array([700, 300], np.int32)
    gw = gpu_workload.GpuWorkload(Workload("pfinf", 512 * KiB, 512 * 200 * KiB,
                                           [ModelSpec("m", FP16, kv_heads, head_dim, 1, kv_heads * group, lens, tag=46)], "shuffle"), zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        m, g = gw.model_ids[0], gw.geom[gw.model_ids[0]]
        off = np.array([0, 700, 1000], np.int32)
        q = torch.randn((1000, kv_heads * group, head_dim), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda", dtype=torch.float16)
        ws = torch.empty(fs.fs_prefill_workspace_bytes(2), dtype=torch.uint8, device="cuda")

        def run():
            out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda")
            fs.fs_prefill_attention(gw.pool, m, 0, kv_heads * group, 0.1, q, gw.tables[0], gw.seq_lens[0], torch.from_numpy(off).cuda(), off, out, lse, ws)
            assert fs.fs_decode_status(ws) == 0 and fs.fs_pool_get_option(gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == kernel
            return out, lse

        out0, lse0 = run()
        T, per_block = g.tokens_per_block, 16 // group
        for t in (5, 61, 133, 690):
            at = int(gw.tables_host[0][0, t // T]) * g.block_budget + g.kv_tile + (t % T) * g.row_bytes  # KV head 0, element 0
            part = gw.pool_mem[at: at + 2]
            old = part.clone()
            part.copy_(torch.tensor([0x00, 0x7C], dtype=torch.uint8))
            out, lse = run()
            part.copy_(old)
            first = t // per_block * per_block
            assert not torch.isfinite(out[t:700, :group, 0]).any(), t
            out[first:700, :group, 0] = out0[first:700, :group, 0]
            assert torch.equal(out, out0) and torch.equal(lse, lse0), t
    finally:
        gw.close()


@pytest.mark.parametrize("dtype,T", [(FP16, 13), (FP16, 16), (INT8, 11), (INT4, 15)])
def test_infinite_last_value_in_large_launches(dtype, T, monkeypatch):
    """An Inf in the sequence's last token (integer formats: in its V scale): its own row is infinite, not NaN, though the
    slots behind it are multiplied with weight 0, and the rows more than a sub-tile in front are what they are without it."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    n, H, group = 700, 2, 4
    par = {FP16: 0, INT8: 2, INT4: 4}[dtype]
    slab = -(-fs.fs_block_bytes(dtype, H, 128, 1, T) // 256) * 256
    gw = gpu_workload.GpuWorkload(Workload("pfinfl", slab, slab * 200, [ModelSpec("m", dtype, H, 128, 1, H * group, np.array([n], np.int32), tag=52,
                                                                                  src_f32=dtype == INT4)], "shuffle"), zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        m, g = gw.model_ids[0], gw.geom[gw.model_ids[0]]
        off = np.array([0, n], np.int32)
        q = torch.randn((n, H * group, 128), generator=torch.Generator(device="cuda").manual_seed(8), device="cuda", dtype=torch.float16)
        ws = torch.empty(fs.fs_prefill_workspace_bytes(1), dtype=torch.uint8, device="cuda")

        def run():
            out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda")
            fs.fs_prefill_attention(gw.pool, m, 0, H * group, 0.1, q, gw.tables[0], gw.seq_lens[0], torch.from_numpy(off).cuda(), off, out, lse, ws)
            assert fs.fs_decode_status(ws) == 0 and fs.fs_pool_get_option(gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) & 0xffff == (16 | 8 << 8)
            return out, lse

        out0, lse0 = run()
        t, tpb = n - 1, g.tokens_per_block
        assert tpb == T
        block = int(gw.tables_host[0][0, t // tpb]) * g.block_budget
        at = block + (g.kv_tile + (t % tpb) * g.row_bytes if dtype == FP16 else 2 * g.kv_tile + g.par_tile + (t % tpb) * par)  # KV head 0
        gw.pool_mem[at: at + 2] = torch.tensor([0x00, 0x7C], dtype=torch.uint8, device="cuda")
        out, lse = run()
        last = out[t, :group, :1 if dtype == FP16 else 128].float()
        # (integers: a code at its zero point is 0 * Inf)
        assert torch.isinf(last).all() if dtype == FP16 else torch.isinf(last).float().mean() > 0.5, last
        out[t // 32 * 32:, :group] = out0[t // 32 * 32:, :group]
        assert torch.equal(out, out0) and torch.equal(lse, lse0)
    finally:
        gw.close()


@pytest.mark.parametrize("head_dim,n_seq,with_tokens,kernel", [(128, 600, 600, 16 | 8 << 8), (256, 300, 300, 4 | 4 << 8), (64, 700, 700, 16 | 8 << 8),
                                                               (128, 100, 100, 8 | 8 << 8), (128, 500, 90, 8 | 8 << 8), (256, 200, 150, 4 | 4 << 8)])
def test_many_sequences(head_dim, n_seq, with_tokens, kernel):
    """More sequences than a workgroup has threads (their tile counts come from the preparation kernel), and direct launches
    whose sequences several waves list, most of them without new tokens."""
    import gpu_harness
    import paper_2509_06261_amd as fs

    rng = np.random.default_rng([head_dim, n_seq])
    lens = rng.integers(1, 40, n_seq).astype(np.int32)
    lens[[0, n_seq // 2, n_seq - 1]] = [150, 97, 33]
    wl = Workload("pfmany", 64 * KiB, 64 * 1500 * KiB, [ModelSpec("m", FP16, 2 if head_dim != 256 else 1, head_dim, 1, 4, lens, tag=47)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[0]])
        n_new = np.minimum(lens, rng.integers(1, 17, n_seq)).astype(np.int32) if with_tokens < 200 else lens.copy()
        n_new[rng.permutation(n_seq)[: n_seq - with_tokens]] = 0
        print(par.prefill_and_check(0, 0, n_new))
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == kernel
    finally:
        par.close()


@pytest.mark.parametrize("kv_heads,n_seq", [(1, 5200), (2, 2500)])
def test_many_items_of_one_or_two_heads(kv_heads, n_seq):
    """Either side of 20 items per compute unit (256 in the card's whole partition), where one or two heads' items are
    ordered head by head and by tile."""
    import gpu_harness

    lens = np.random.default_rng(n_seq).integers(1, 4, n_seq).astype(np.int32)
    lens[[7, n_seq - 3]] = [70, 33]
    wl = Workload("pf1h", 8 * KiB, 8 * KiB * (n_seq + 100), [ModelSpec("m", FP16, kv_heads, 128, 1, 4, lens, tag=57)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[0]])
        print(par.prefill_and_check(0, 0, lens))
    finally:
        par.close()


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,kv_heads,group", [(64, 6, 4), (128, 2, 4), (128, 3, 1)])
def test_small_launches(dtype, head_dim, kv_heads, group):
    """Launches with no more items than compute units: no preparation kernel, items of half the size, exact codes."""
    import gpu_harness
    import paper_2509_06261_amd as fs

    wl = Workload("pfsm", 384 * KiB, 384 * 200 * KiB,
                  [ModelSpec("m", dtype, kv_heads, head_dim, 2, kv_heads * group, EDGES, tag=43, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[1]])
        n_new = EDGES if head_dim == 128 else np.minimum(EDGES, 40)
        print(par.prefill_and_check(0, 1, n_new), par.prefill_and_check(0, 1, np.minimum(EDGES, CHUNKS)))
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (8 | 8 << 8)
    finally:
        par.close()


def _groups(pool):
    """log2 of the groups of waves that the latest launch may deal contexts to; the kernel is that of the small launches."""
    import paper_2509_06261_amd as fs

    assert fs.fs_pool_get_option(pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (8 | 8 << 8)
    items = fs.fs_pool_get_option(pool, fs.FS_OPT_LAST_PREFILL_ITEMS)
    assert items & 255 == (4 if items >> 8 == 2 else 8), items
    return items >> 8


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,kv_heads,group,n_new,shift", [(128, 8, 4, [100, 16, 0, 70], 2), (128, 8, 1, [33, 200, 40, 5], 2), (128, 6, 4, [300, 40, 40, 1], 2),
                                                                 (64, 16, 4, [64, 17, 40, 3], 2), (64, 12, 8, [90, 30, 40, 33], 1), (128, 12, 8, [90, 30, 40, 33], 1)])
def test_context_groups(dtype, head_dim, kv_heads, group, n_new, shift):
    """Small launches behind long contexts: two and four groups of waves per context (items of 8 and 4 blocks), sequences
    of less than a step, a group without tokens, ragged items."""
    import gpu_harness

    lens = np.array([1500 if shift == 2 else 2060, 1111, 40, 260], np.int32)
    wl = Workload("pfgrp", 160 * KiB, 160 * 600 * KiB, [ModelSpec("m", dtype, kv_heads, head_dim, 1, kv_heads * group, lens, tag=50, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[0]])
        print(par.prefill_and_check(0, 0, np.array(n_new, np.int32)))
        assert _groups(par.gw.pool) == shift
    finally:
        par.close()


@pytest.mark.parametrize("dtype,T,shift", [(FP16, 9, 2), (INT8, 13, 2), (INT4, 60, 2), (FP16, 13, 1), (FP8, 9, 1), (INT4, 11, 1), (FP16, 13, 0), (FP8, 9, 0),
                                           (INT8, 11, 0), (INT4, 60, 0)])
def test_several_table_segments_of_odd_blocks(dtype, T, shift, monkeypatch):
    """Contexts of two and three table segments whose blocks are no multiple of eight tokens: segments that begin inside a
    block, the refilled table, the last segment's end; in two and four groups of waves and in the 16-block kernel (0)."""
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    if shift == 0:
        monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    segment = min(500 * T // 128 * 128, 8192)
    # (two groups: one new token more than four blocks hold in every sequence, tiles enough for every unit but in halves)
    lens, n_new, heads, group = {0: ([2 * segment + 77, segment + 1], [70, 33], 2, 4), 1: ([2 * segment + 77, segment + 3] + [40] * 15, [5] * 17, 8, 9),
                                 2: ([2 * segment + 77, segment + 1], [40, 18], 4, 4)}[shift]
    lens = np.array(lens, np.int32)
    slab = -(-fs.fs_block_bytes(dtype, heads, 128, 1, T) // 256) * 256
    wl = Workload("pfseg", slab, slab * int((-(-lens // T)).sum() + 20),
                  [ModelSpec("m", dtype, heads, 128, 1, heads * group, lens, tag=54, src_f32=dtype == INT4)], "shuffle")
    p = gpu_harness.Parity(wl, zero_pool=True)
    try:
        assert p.gw.T[p.gw.model_ids[0]] == T
        p.gw.populate([[0]])
        print(p.prefill_and_check(0, 0, np.array(n_new, np.int32)))
        assert _groups(p.gw.pool) == shift if shift else fs.fs_pool_get_option(p.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) & 0xffff == (16 | 8 << 8)
    finally:
        p.close()


def test_contexts_are_dealt_to_groups_by_their_lengths():
    """A chunk behind 3000 tokens: its kernel has groups of waves and uses them (other roundings than the walk without, which
    the same chunk takes among more sequences than a workgroup lists)."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    n_new, H, group = 40, 8, 4
    gw = gpu_workload.GpuWorkload(Workload("pfdeal", 256 * KiB, 256 * 300 * KiB, [ModelSpec("m", FP16, H, 128, 1, H * group, np.array([3000], np.int32), tag=55)], "shuffle"),
                                  zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        q = torch.randn((n_new, H * group, 128), generator=torch.Generator(device="cuda").manual_seed(10), device="cuda", dtype=torch.float16)
        got = []
        for n_seq, groups in ((1, 2), (600, 0)):
            off = np.full(n_seq + 1, n_new, np.int32)
            off[0] = 0
            ws = torch.empty(fs.fs_prefill_workspace_bytes(n_seq), dtype=torch.uint8, device="cuda")
            table, lens = gw.tables[0].repeat(n_seq, 1), gw.seq_lens[0].repeat(n_seq)
            out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda")
            fs.fs_prefill_attention(gw.pool, gw.model_ids[0], 0, H * group, 0.1, q, table, lens, torch.from_numpy(off).cuda(), off, out, lse, ws)
            assert fs.fs_decode_status(ws) == 0 and _groups(gw.pool) == groups
            got.append(out.float())
        # (values of N(0, 1) averaged: below 4, so two results each within 2^-11 of a weight's rounding and the output's)
        diff = (got[0] - got[1]).abs().max().item()
        assert 0 < diff < 2 * 4 * 2.0 ** -10, diff
    finally:
        gw.close()


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("head_dim,kv_heads,lens,n_new", [(128, 8, [777], [777]), (128, 8, [400, 63], [400, 63]), (64, 16, [500], [300]),
                                                          (128, 4, [880, 40], [40, 7]), (128, 1, [150] + [30] * 99, [60] + [30] * 99)])
def test_short_contexts_behind_a_wide_table(dtype, head_dim, kv_heads, lens, n_new):
    """Short prompts and chunks take the walk without groups of waves however long a context the table could hold: the very
    results of the same call over a table that just fits."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    lens, n_new, group = np.array(lens, np.int32), np.array(n_new, np.int32), 4
    slab = kv_heads * head_dim * 2 * 70  # 35 to 140 tokens
    gw = gpu_workload.GpuWorkload(Workload("pfwide", slab, slab * 400, [ModelSpec("m", dtype, kv_heads, head_dim, 1, kv_heads * group, lens, tag=53,
                                                                                          src_f32=dtype == INT4)], "shuffle"), zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        m, T = gw.model_ids[0], gw.geom[gw.model_ids[0]].tokens_per_block
        off = np.concatenate([[0], np.cumsum(n_new)]).astype(np.int32)
        q = torch.randn((int(off[-1]), kv_heads * group, head_dim), generator=torch.Generator(device="cuda").manual_seed(9), device="cuda", dtype=torch.float16)
        ws = torch.empty(fs.fs_prefill_workspace_bytes(len(lens)), dtype=torch.uint8, device="cuda")
        narrow = gw.tables[0].contiguous()
        wide = torch.zeros((len(lens), 32768 // T), dtype=torch.int32, device="cuda")
        wide[:, : narrow.shape[1]] = narrow
        assert narrow.shape[1] * T < 1024
        got = []
        for table in (narrow, wide):
            out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda")
            fs.fs_prefill_attention(gw.pool, m, 0, kv_heads * group, 0.1, q, table, gw.seq_lens[0], torch.from_numpy(off).cuda(), off, out, lse, ws)
            assert fs.fs_decode_status(ws) == 0 and fs.fs_pool_get_option(gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (8 | 8 << 8)
            got.append((out, lse))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        assert bool(got[0][0].ne(0).any(-1).all())
    finally:
        gw.close()


@pytest.mark.parametrize("head_dim,kv_heads,length,shift", [(128, 8, 1400, 2), (64, 24, 1400, 2), (128, 48, 2200, 1)])
def test_infinite_value_with_context_groups(head_dim, kv_heads, length, shift):
    """The rows of blocks in front of the token that holds an Inf are what they are without it, with groups of waves too."""
    import torch

    import gpu_workload
    import paper_2509_06261_amd as fs

    lens, n_new, group = np.array([length], np.int32), 90, 4
    gw = gpu_workload.GpuWorkload(Workload("pfgi", 512 * KiB, 512 * 200 * KiB,
                                           [ModelSpec("m", FP16, kv_heads, head_dim, 1, kv_heads * group, lens, tag=51)], "shuffle"), zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        m, g = gw.model_ids[0], gw.geom[gw.model_ids[0]]
        off = np.array([0, n_new], np.int32)
        q = torch.randn((n_new, kv_heads * group, head_dim), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda", dtype=torch.float16)
        ws = torch.empty(fs.fs_prefill_workspace_bytes(1), dtype=torch.uint8, device="cuda")

        def run():
            out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], device="cuda")
            fs.fs_prefill_attention(gw.pool, m, 0, kv_heads * group, 0.1, q, gw.tables[0], gw.seq_lens[0], torch.from_numpy(off).cuda(), off, out, lse, ws)
            assert fs.fs_decode_status(ws) == 0 and _groups(gw.pool) == shift
            return out, lse

        out0, lse0 = run()
        T = g.tokens_per_block
        for t in (length - 89, length - 63, length - 2):
            at = int(gw.tables_host[0][0, t // T]) * g.block_budget + g.kv_tile + (t % T) * g.row_bytes  # KV head 0, element 0
            part = gw.pool_mem[at: at + 2]
            old = part.clone()
            part.copy_(torch.tensor([0x00, 0x7C], dtype=torch.uint8))
            out, lse = run()
            part.copy_(old)
            row = t - (length - n_new)
            assert not torch.isfinite(out[row:, :group, 0]).any(), t
            out[row // 4 * 4:, :group, 0] = out0[row // 4 * 4:, :group, 0]
            assert torch.equal(out, out0) and torch.equal(lse, lse0), t
    finally:
        gw.close()


@pytest.mark.parametrize("dtype", [FP16, FP8, INT8, INT4])
@pytest.mark.parametrize("group,lens,seqs", [(16, [96] * 40 + [97, 1, 95, 33, 130, 240, 385, 500], [0, 40, 41, 42, 43, 44]), (4, [480] * 12 + [500, 97, 130, 1], [12, 13, 14, 15])])
def test_large_launches_at_head_dim_64(dtype, group, lens, seqs):
    """Items of 32 and 24 blocks: at least eight of them per compute unit (256 in the card's whole partition).  (With 16 query heads
    per KV head the oracle would take most of a minute over the three longest sequences; with four it does the longest.)"""
    import gpu_harness
    import paper_2509_06261_amd as fs

    lens = np.array(lens, np.int32)
    wl = Workload("pf64w", 192 * KiB, 192 * 900 * KiB, [ModelSpec("m", dtype, 40, 64, 1, 40 * group, lens, tag=49, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        par.gw.populate([[0]])
        print("T", par.gw.T, par.prefill_and_check(0, 0, lens, seqs=np.array(seqs)))
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (16 | 8 << 8)
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_ITEMS) == (32 if dtype == FP16 else 24)
    finally:
        par.close()


@pytest.mark.parametrize("dtype,T,head_dim,heads,group,large", [(FP16, 13, 128, 2, 4, 1), (FP8, 9, 128, 2, 1, 1), (INT8, 31, 128, 2, 4, 1),
                                                                (INT4, 11, 128, 2, 4, 1), (INT4, 61, 128, 2, 1, 0), (INT8, 8, 128, 3, 4, 0),
                                                                (FP8, 250, 64, 16, 4, 1), (INT4, 15, 64, 16, 4, 1), (FP16, 9, 256, 4, 4, 1)])
def test_blocks_of_any_token_count(dtype, T, head_dim, heads, group, large, monkeypatch):
    """Sub-tiles of 32 tokens over blocks that end anywhere: rows of eight tokens from two blocks, the last block's end."""
    import gpu_harness
    import gpu_workload
    import paper_2509_06261_amd as fs

    if large and head_dim == 128:
        monkeypatch.setattr(gpu_workload, "DEFAULT_OPTIONS", {fs.FS_OPT_PREFILL_COLUMN_BLOCKS: 16})
    slab = -(-fs.fs_block_bytes(dtype, heads, head_dim, 1, T) // 256) * 256
    wl = Workload("pftok", slab, slab * 600, [ModelSpec("m", dtype, heads, head_dim, 1, heads * group, EDGES, tag=48, src_f32=dtype == INT4)], "shuffle")
    par = gpu_harness.Parity(wl, zero_pool=True)
    try:
        assert par.gw.T[par.gw.model_ids[0]] == T
        par.gw.populate([[0]])
        print("T", par.gw.T, par.prefill_and_check(0, 0, EDGES), par.prefill_and_check(0, 0, np.minimum(EDGES, CHUNKS)))
        assert fs.fs_pool_get_option(par.gw.pool, fs.FS_OPT_LAST_PREFILL_KERNEL) >> 8 & 255 in (4, 8) or head_dim == 256
    finally:
        par.close()


def test_small_launch_reports_and_follows_no_bad_entry():
    """The status word of a launch without preparation: 0 for a good call whatever the workspace held, bit 0 for a length
    or chunk out of range, bit 2 for a block-table entry outside the pool -- inside a sequence with new tokens only."""
    import torch

    import paper_2509_06261_amd as fs

    slab, n_slabs, lens = 64 * KiB, 64, [40, 200, 90]
    mem = torch.zeros(slab * n_slabs, dtype=torch.uint8, device="cuda")
    pool = fs.fs_pool_create(slab, mem.numel(), mem)
    try:
        _, model = fs.fs_model_register(pool, fs.FS_KV_FP16, 2, 128, 1)
        T = fs.fs_model_geometry(pool, model).tokens_per_block
        table = np.full((3, -(-max(lens) // T)), -1, np.int32)
        for i, n in enumerate(lens):
            table[i, : -(-n // T)] = fs.fs_blocks_alloc(pool, model, -(-n // T))[1]
        table[2, 0] = -1  # sequence 2 brings no tokens: its entries are not read

        def status(lens, table, offsets):
            off = np.array(offsets, np.int32)
            q = torch.ones((int(off[-1]), 8, 128), dtype=torch.float16, device="cuda")
            ws = torch.full((fs.fs_prefill_workspace_bytes(3),), 0xff, dtype=torch.uint8, device="cuda")
            fs.fs_prefill_attention(pool, model, 0, 8, 0.1, q, torch.from_numpy(table).cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda"),
                                    torch.from_numpy(off).cuda(), off, torch.empty_like(q), None, ws)
            torch.cuda.synchronize()
            assert fs.fs_pool_get_option(pool, fs.FS_OPT_LAST_PREFILL_KERNEL) == (8 | 8 << 8)
            return fs.fs_decode_status(ws)

        assert status(lens, table, [0, 40, 240, 240]) == 0
        assert status([30, 200, 90], table, [0, 40, 240, 240]) == 1
        bad = table.copy()
        bad[1, 0] = 1 << 20
        assert status(lens, bad, [0, 40, 41, 41]) == 4
        assert status([0, 200, 90], bad, [0, 40, 41, 41]) == 5
    finally:
        fs.fs_pool_destroy(pool)
