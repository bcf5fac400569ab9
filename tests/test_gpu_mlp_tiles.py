"""The surrogate network's kernels at the edges of their tiles: 16 rows per
workgroup, 512 workgroups per pass, 256 rows per step of the gradient
reductions, 65 536 rows per trip of a prediction."""

import numpy as np
import pytest

from oracle import mlp
from paper_2609_21204_amd import dybond as db

pytestmark = pytest.mark.gpu


def _data(seed, n):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1.0, 1.0, (n, 4)).astype(np.float32)
    return x, rng.uniform(0.0, 1.0, (n, 2)).astype(np.float32)


@pytest.mark.parametrize("n", [1, 16, 17, 8192, 8193, 65536, 65553])
def test_predict_gives_each_row_its_own_output(n):
    x, _ = _data(n, n)
    h = db.db_mlp_create(64)
    try:
        params = mlp.init_params(3)
        db.db_mlp_set_params(h, params)
        y = db.db_mlp_predict(h, x)
        # a row's output does not depend on the rows beside it
        pick = np.unique(np.clip([0, 15, 16, n // 2, 8191, 8192, 65535, 65536, n - 1], 0, n - 1))
        alone = np.concatenate([db.db_mlp_predict(h, x[k:k + 1]) for k in pick])
    finally:
        db.db_mlp_destroy(h)
    assert np.array_equal(y[pick], alone)
    # FP32 against FP64, with one bf16 rounding (2^-8) of an activation next
    # to a rounding boundary allowed for
    assert np.max(np.abs(y[pick] - mlp.forward(params, x[pick])[0])) < 1e-3


@pytest.mark.parametrize("n", [1, 16, 255, 256, 257, 512, 513, 1000])
def test_gradients_at_the_edges_of_the_reductions(n):
    x, t = _data(n + 7, n)
    h = db.db_mlp_create(1000)
    try:
        params = mlp.init_params(n)
        db.db_mlp_set_params(h, params)
        loss, g = db.db_mlp_loss_grad(h, x, t)
    finally:
        db.db_mlp_destroy(h)
    l_ref, g_ref = mlp.loss_and_grad(params, x, t)
    assert abs(loss - l_ref) <= 1e-4 * l_ref + 1e-9
    k = 0
    for name, shape in mlp.SHAPES:
        size = int(np.prod(shape))
        a, b = g[k:k + size], g_ref[k:k + size]
        # a bf16 rounding the other way moves one product by 2^-8 of itself;
        # over few rows that is up to 2^-8 of a gradient
        assert np.max(np.abs(a - b)) <= 2.0 ** -8 * np.max(np.abs(b)) + 1e-8, name
        k += size
