"""Every device call of the binding runs on torch's current stream, through the native marshaling as through ctypes: on a stream
of their own, behind a kernel that keeps that stream busy, the calls see what the stream brings before them and nothing else."""
import numpy as np
import pytest

from fs_inputs.workloads import FP16, KiB, ModelSpec, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("kind", ["append", "append_multi", "decode", "decode_multi", "decode_step", "prefill"])
def test_calls_run_on_the_current_stream(kind, native, monkeypatch):
    import torch

    import gpu_workload
    from paper_2509_06261_amd import binding as fs

    lens, H, D, group = np.array([40, 100, 7], np.int32), 4, 64, 2
    n, heads = len(lens), H * group
    gw = gpu_workload.GpuWorkload(Workload("strm", 32 * KiB, 32 * 64 * KiB, [ModelSpec("m", FP16, H, D, 1, heads, lens, tag=56)], "shuffle"), zero_pool=True)
    try:
        gw.place()
        gw.populate([[0]])
        fs._slow()  # (CUDA is up: the next calls are marshaled natively)
        if not native:
            monkeypatch.setattr(fs, "_fast", fs._NotYet)
            monkeypatch.setattr(fs, "_slow", lambda: None)
        elif fs._fast is fs._NotYet:
            pytest.fail("the native marshaling did not come up")
        m, table, seq_lens = gw.model_ids[0], gw.tables[0], gw.seq_lens[0]
        rows = n if kind != "prefill" else int(lens.sum())
        gen = torch.Generator(device="cuda").manual_seed(11)
        new = [torch.randn(shape, generator=gen, device="cuda", dtype=torch.float16) for shape in ((rows, heads, D), (n, H, D), (n, H, D))]
        q, k, v = [torch.zeros_like(x) for x in new]
        out, lse = torch.zeros_like(q), torch.zeros((rows, heads), device="cuda")
        seq_idx, pos = torch.arange(n, dtype=torch.int32, device="cuda"), (seq_lens - 1).to(torch.int32)
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        off_d = torch.from_numpy(off).cuda()
        batch, append = fs.make_batch(m, 0, heads, 0.1, q, table, seq_lens, out, lse, lens), fs.make_append(m, 0, k, v, seq_idx, pos, table)
        ws = torch.empty(max(fs.fs_prefill_workspace_bytes(n), fs.fs_decode_workspace_bytes(gw.pool, [batch])), dtype=torch.uint8, device="cuda")

        def call():
            if kind == "append":
                fs.fs_kv_append(gw.pool, m, 0, k, v, seq_idx, pos, table)
            elif kind == "append_multi":
                fs.fs_kv_append_multi(gw.pool, [append])
            elif kind == "decode":
                fs.fs_decode_attention(gw.pool, m, 0, heads, 0.1, q, table, seq_lens, out, lse, ws)
            elif kind == "decode_multi":
                fs.fs_decode_attention_multi(gw.pool, [batch], ws)
            elif kind == "decode_step":
                fs.fs_decode_step_multi(gw.pool, [append], [batch], ws)
            else:
                fs.fs_prefill_attention(gw.pool, m, 0, heads, 0.1, q, table, seq_lens, off_d, off, out, lse, ws)

        def results():
            return [x.clone() for x in (out, lse, gw.pool_mem)]

        def bring():
            for x, y in zip((q, k, v), new):
                x.copy_(y)

        start = gw.pool_mem.clone()
        bring()
        call()
        torch.cuda.synchronize()
        want = results()
        gw.pool_mem.copy_(start)
        for x in (q, k, v, out, lse):
            x.zero_()
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            torch.cuda._sleep(100_000_000)  # some 50 milliseconds
            bring()
            call()
        assert not side.query()  # (the call did not wait for the stream)
        side.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(results(), want)), kind
        assert not torch.equal(want[0], torch.zeros_like(want[0])) or kind.startswith("append")
    finally:
        gw.close()
