"""How much workspace the history of omega may take (4 k n bytes): none of it
where it would be over 4 GiB, or over both a quarter of A and 16 MiB, or would
push a problem that fits the static entry point's array out of it."""
import pytest

import paper_1312_6838_amd as g


def _bytes(m, n, k):
    return g.workspace_size(g.make_desc(m, n, m, g.F32, 1 << 20, None, k, 16, False, 0.0, None))


@pytest.mark.parametrize("m,n,k,kept", [
    (2048, 1 << 24, 63, True),      # 3.9 GiB of 128
    (2048, 1 << 24, 65, False),     # 4.1 GiB
    (1024, 1 << 18, 256, False),    # a quarter of A, but the rest fits the static array
    (1024, 1 << 18, 257, False),
    (1024, 1 << 22, 256, True),     # a quarter of A and 4 GiB
    (1024, 1 << 22, 257, False),
    (1024, 1 << 21, 256, True),     # a quarter of A
    (1024, 1 << 21, 257, False),
    (64, 1 << 20, 4, True),         # 16 MiB
    (64, 1 << 20, 17, False),       # over a quarter (16 columns' worth) and 16 MiB
])
def test_history_share_of_the_workspace(m, n, k, kept):
    # the rest that grows with k (basis, step vectors) is far below 4 k n here
    per_column = (_bytes(m, n, k) - _bytes(m, n, 1)) / n
    if kept:
        assert 4 * (k - 1) - 1 <= per_column <= 4 * (k - 1) + 60
    else:
        assert per_column <= 60 - 4
