"""Lists of one row straight from the pattern flags: rows around the pieces of eight keys and the spans of 2048 keys that the
kernels work in, flag rows of odd length (so of every alignment), rows inside and below a true-mask block."""
import numpy as np
import pytest

from test_gpu_decode import group_lists_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,H,S,L,rows", [
    (1, 3, 4101, 0, (0, 6, 7, 8, 2047, 2048, 2049, 4095, 4096, 4100)), (4, 8, 6151, 0, (2046, 2055, 6150)),
    (8, 8, 2049, 0, (2048,)), (2, 6, 333, 203, (195, 199, 202, 203, 210, 211, 332)),
])
def test_rows_around_pieces_and_spans(G, H, S, L, rows):
    rng = np.random.default_rng(S + G)
    dflag, vflag = ((rng.random((H, S)) < 0.03).astype(np.uint8) for _ in range(2))
    for h in range(H):
        dflag[h, : 5 * h] = 1
        vflag[h, -3:] = 1
    tm = np.tril(rng.random((H, L, L)) < 0.3).astype(np.uint8) if L else None
    for row in rows:
        group_lists_case(H, G, S, row, dflag, vflag, **({"L": L, "true_mask": tm} if L else {}))
