"""The workspace of a batch serves every smaller batch too: sequences leave, and the library is asked once."""
import pytest

import tidar_inputs as TI


@pytest.mark.parametrize("d,ff,heads,kv,k", [(5760, 11008, 40, 8, 8), (4096, 12288, 32, 8, 8), (2176, 5632, 16, 4, 4),
                                             (1536, 8960, 12, 2, 8), (4096, 12288, 32, 1, 4), (4096, 12288, 32, 8, 1)])
def test_one_more_sequence_never_needs_less(d, ff, heads, kv, k):
    import paper_2511_08923_amd as T
    ctx = T.tidar_create(T.make_config(TI.ModelShape("t", 2, d, heads, kv, 128, ff, 32000, False), T.TIDAR_BF16, max_k=16, max_batch=64))
    sizes = [T.tidar_workspace_bytes(ctx, b, k, 4096) for b in range(1, 65)]
    T.tidar_destroy(ctx)
    assert all(x <= y for x, y in zip(sizes, sizes[1:])), [b + 1 for b, (x, y) in enumerate(zip(sizes, sizes[1:])) if x > y]
