"""The network's tanh.  Inference rounds tanh to bfloat16 from the hardware's
exponential and reciprocal wherever their error cannot change the rounding;
training takes tanhf.  Both have to give the same bits: every float through
the fast path beside tanhf, and the two forward passes beside each other."""
import ctypes as C
import os

import numpy as np
import pytest

import build_checks
from paper_2605_07083_amd import presets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sweep():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    if not os.path.exists(build_checks.TANH_SWEEP):
        build_checks.build()
    f = C.CDLL(build_checks.TANH_SWEEP).tanh_sweep
    f.argtypes, f.restype = [C.c_uint32, C.c_ulonglong, C.POINTER(C.c_ulonglong)], C.c_int
    return f


@pytest.mark.parametrize("quarter", range(4))
def test_every_float_rounds_as_tanhf_does(sweep, quarter):
    """All 2^32 floats (both signs, zeros, denormals, infinities, NaNs): where
    the interval's ends agree they are bf16(tanhf(x)), and after tanhf has
    decided the others every value is.  Each quarter holds values that the
    interval decides (from about 1e-4 on it decides nearly all)."""
    print("case: tanh of the floats from 0x%08x on" % (quarter << 30), flush=True)
    out = (C.c_ulonglong * 4)()
    assert sweep(quarter << 30, 1 << 28, out) == 0
    closed, closed_wrong, settled_wrong, a_wrong = list(out)
    print("  decided by the interval %.6f, wrong %d (one: 0x%08x), after tanhf wrong %d"
          % (closed / 2.0 ** 30, closed_wrong, a_wrong, settled_wrong), flush=True)
    assert closed > 0 and closed_wrong == 0 and settled_wrong == 0


# seeds and shapes: one tile and ragged ones, weights up to saturating every tanh
@pytest.mark.parametrize("B,X,scale", [(1, 64, 1.0), (3, 320, 1.0), (8, 704, 3.0), (16, 2048, 1.0), (4, 1216, 0.05)])
def test_training_and_inference_forward_passes_agree(sweep, B, X, scale):
    """The training step's loss against the inference pass's own output is
    zero: no output differs in any bit."""
    import torch
    from paper_2605_07083_amd import surrogate as sur
    print("case: training against inference, B=%d X=%d scale %g" % (B, X, scale), flush=True)
    W, b = presets.surrogate_test_weights(51 + B, scale)
    net = sur.Surrogate(B, X, device="cuda:0")
    q = presets.surrogate_params(B, 53)
    p = torch.tensor(np.stack([q["gamma_emit"], q["T_K"], q["V"], q["ng"]], 1), dtype=torch.float32, device="cuda:0")
    net.set_weights(W, b)
    out = net.forward(p)
    assert float(out.abs().max()) > 0.0
    assert net.train_step(p, out, 1e-3) == 0.0
    net.close()
