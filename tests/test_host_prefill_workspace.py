"""The two sizes of a prefill workspace (no GPU needed): with room for the pieces of split items, and the least that is accepted."""
import pytest

import paper_2509_06261_amd as fs


@pytest.mark.parametrize("n_seq", [1, 2, 64, 512, 513, 4096, 1 << 20])
def test_least_workspace(n_seq):
    least, full = fs.fs_prefill_least_workspace_bytes(n_seq), fs.fs_prefill_workspace_bytes(n_seq)
    assert least % 256 == 0 and 4 * (n_seq + 1) < least <= 4 * n_seq + 9216
    assert full - least == 8 * 256 + 512 * 133120  # counters and two places for each of 256 workgroups
    # a workspace sized for more sequences does for fewer
    assert least <= fs.fs_prefill_least_workspace_bytes(n_seq + 1) and full <= fs.fs_prefill_workspace_bytes(n_seq + 1)


def test_no_sequences():
    assert fs.fs_prefill_least_workspace_bytes(0) == fs.fs_prefill_workspace_bytes(0) == 0
