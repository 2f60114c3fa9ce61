"""Order of surrogate calls on streams whose handles have the same value: hipStreamPerThread names
another stream in every thread, and a destroyed stream's address may be given to the next one."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PER_THREAD = 2          # hipStreamPerThread


def hip():
    return ctypes.CDLL(None)      # the process's own HIP runtime, loaded with the library


def _setup():
    import torch
    from paper_2009_10400_amd import surrogate
    rng = np.random.default_rng(4)
    x, p, t = (torch.from_numpy(rng.uniform(-1, 1, (3000, k)).astype(np.float32)).to("cuda:0") for k in (3, 3, 4))
    ref, mlp = (surrogate.MLP(0, n_param=3, n_freq=16, width=128, depth=3, n_out=4, seed=3) for _ in range(2))
    for m in (ref, mlp):                     # workspaces are there before the streams are busy
        m.gradient(x, p, t)
    torch.cuda.synchronize()
    return torch, surrogate, ref, mlp, x, p, t


def _on(surrogate, mlp, stream, fn, *args):
    lib = surrogate._lib
    assert lib.tled_mlp_begin(mlp._h, ctypes.c_void_p(stream)) == 0
    try:
        assert fn(mlp._h, *args) == 0
    finally:
        assert lib.tled_mlp_end(mlp._h) == 0


def test_per_thread_streams_of_two_threads():
    torch, surrogate, ref, mlp, x, p, t = _setup()
    lib, dp = surrogate._lib, surrogate._dp
    out = torch.zeros((3000, 4), dtype=torch.float32, device="cuda:0")
    torch.cuda.synchronize()
    src = torch.empty(64 << 20, dtype=torch.float32, device="cuda:0")
    big = torch.empty_like(src)
    torch.cuda.synchronize()
    for k in range(3):
        ref.train_step(x, p, t, 1e-2)
        want = ref.forward(x, p).cpu().numpy()
        enqueued, leave = threading.Event(), threading.Event()

        def train():
            # long enough for the other thread's forward pass to overtake it if nothing orders the two
            for _ in range(40):
                lib.tled_stream_copy(0, dp(big), dp(src), big.numel() * 4, ctypes.c_void_p(PER_THREAD))
            _on(surrogate, mlp, PER_THREAD, lib.tled_mlp_train_step, 3000, dp(x), dp(p), dp(t), 1e-2, None)
            enqueued.set()
            leave.wait(60)

        th = threading.Thread(target=train, daemon=True)
        th.start()
        enqueued.wait(60)
        _on(surrogate, mlp, PER_THREAD, lib.tled_mlp_forward, 3000, dp(x), dp(p), dp(out))
        status = hip().hipStreamSynchronize(ctypes.c_void_p(PER_THREAD))
        leave.set()
        th.join()
        assert status == 0
        assert np.array_equal(out.cpu().numpy(), want), k
        torch.cuda.synchronize()


def test_streams_created_and_destroyed_between_the_calls():
    torch, surrogate, ref, mlp, x, p, t = _setup()
    lib, dp = surrogate._lib, surrogate._dp
    out = torch.zeros((3000, 4), dtype=torch.float32, device="cuda:0")
    src = torch.empty(64 << 20, dtype=torch.float32, device="cuda:0")
    big = torch.empty_like(src)
    torch.cuda.synchronize()
    for k in range(4):
        ref.train_step(x, p, t, 1e-2)
        want = ref.forward(x, p).cpu().numpy()
        torch.cuda.synchronize()
        a, b = ctypes.c_void_p(), ctypes.c_void_p()
        assert hip().hipStreamCreateWithFlags(ctypes.byref(a), 1) == 0       # hipStreamNonBlocking
        for _ in range(40):
            lib.tled_stream_copy(0, dp(big), dp(src), big.numel() * 4, a)
        _on(surrogate, mlp, a.value, lib.tled_mlp_train_step, 3000, dp(x), dp(p), dp(t), 1e-2, None)
        assert hip().hipStreamDestroy(a) == 0
        assert hip().hipStreamCreateWithFlags(ctypes.byref(b), 1) == 0
        _on(surrogate, mlp, b.value, lib.tled_mlp_forward, 3000, dp(x), dp(p), dp(out))
        assert hip().hipStreamSynchronize(b) == 0
        assert hip().hipStreamDestroy(b) == 0
        assert np.array_equal(out.cpu().numpy(), want), k
