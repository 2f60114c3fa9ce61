"""Calls between tled_mlp_begin and tled_mlp_end that do not fit: refused, without a deadlock and with the
handle as usable as before; parameters may be read and written in between."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(60)
def test_begin_and_end_that_do_not_pair():
    import torch
    from paper_2009_10400_amd import surrogate, tled
    lib, fp = surrogate._lib, surrogate._fp
    mlp = surrogate.MLP(0, n_param=3, n_freq=16, width=64, depth=2, n_out=4, seed=3)
    rng = np.random.default_rng(2)
    x, p = (torch.from_numpy(rng.uniform(-1, 1, (100, 3)).astype(np.float32)).to("cuda:0") for _ in range(2))
    want, theta = mlp.forward(x, p).cpu().numpy(), mlp.params()
    stream = ctypes.c_void_p(torch.cuda.current_stream(0).cuda_stream)
    assert lib.tled_mlp_end(mlp._h) == tled.E_STATE
    assert lib.tled_mlp_begin(mlp._h, stream) == 0
    assert lib.tled_mlp_begin(mlp._h, stream) == tled.E_STATE
    assert lib.tled_mlp_set_stream(mlp._h, None) == tled.E_STATE
    got = np.zeros_like(theta)
    assert lib.tled_mlp_get_params(mlp._h, got.ctypes.data_as(fp)) == 0 and np.array_equal(got, theta)
    assert lib.tled_mlp_set_params(mlp._h, theta.ctypes.data_as(fp)) == 0
    other = []
    th = threading.Thread(target=lambda: other.append(lib.tled_mlp_end(mlp._h)))
    th.start()
    th.join()
    assert other == [tled.E_STATE]
    assert lib.tled_mlp_end(mlp._h) == 0
    assert lib.tled_mlp_end(mlp._h) == tled.E_STATE
    assert np.array_equal(mlp.forward(x, p).cpu().numpy(), want)
