"""Stage-1 scoring with 16- and 32-token sets per wave, at the workgroup counts
where the choice changes, and the ranking of scores that agree in their top 32
bits (tiles of the same tokens in another order, whose means differ in the
last bits, and equal tiles): keys, scores, order and u against the oracle,
bit for bit."""
import numpy as np
import pytest

import synth
from oracle import rift_oracle as O
from tests.rift_testlib import f64, upload
from tests.test_gpu_stages import R, check_stage1, run_score  # noqa: F401  (R: the fixture)

pytestmark = pytest.mark.gpu


# 32-token sets of n_v = 40 or 33 tokens: two a tile, four a workgroup
@pytest.mark.parametrize("dtype,n_tiles,n_v,d", [
    ("bf16", 256, 40, 64), ("bf16", 257, 40, 64), ("bf16", 512, 33, 32), ("bf16", 513, 33, 32), ("bf16", 768, 40, 288),
    ("bf16", 770, 40, 32), ("f32", 256, 33, 64), ("f32", 258, 33, 64), ("f32", 770, 20, 32)])
def test_token_sets_and_close_scores(R, dtype, n_tiles, n_v, d):  # noqa: F811
    rng = np.random.default_rng(n_tiles + d)
    x = rng.standard_normal((n_tiles, n_v, d)).astype(np.float32)
    for t in range(8, n_tiles, 3):
        x[t] = x[t % 7][rng.permutation(n_v)]     # same tokens, another order
    x[5] = x[n_tiles - 1] = x[2]                  # equal tiles
    q = rng.standard_normal((4, d))
    q = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32)
    X, Q = synth.store(x, dtype), synth.store(q, dtype)
    X64, Q64 = f64(X, dtype), f64(Q, dtype)
    ref = O.scene_query_stage1(X64, Q64, 0, 0.4)
    check_stage1(run_score(R, upload(X, dtype), upload(Q, dtype), 0, 0.4), ref, X64, Q64)
