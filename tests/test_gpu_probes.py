"""The product probes run the arithmetic that the kernels use, with the right words."""
import ctypes

import pytest
import torch

from gpu_util import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("log_n,ell", [(3, 1), (13, 6)])
def test_probe_products(kind, log_n, ell):
    # thread t's word is the sum over its chains c of (8t + c + 1) * w^iters modulo the first
    # Q prime (kind 0) or P prime
    import paper_2603_16692_amd as ks
    G = ks.KsParams(1, log_n, ell)
    q = G.moduli[0 if kind == 0 else G.ell]
    w, blocks, iters, chains = q // 3 + 1, 3, 50, ks.raw_call("ks_modmul_chains")
    sink = torch.zeros(blocks * 256, dtype=torch.int64, device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert ks.raw_call("ks_modmul_rate", G._h, kind, blocks, iters, ctypes.c_void_p(sink.data_ptr()), stream) == 0
    wp = pow(w, iters, q)
    want = [sum((chains * t + c + 1) * wp for c in range(chains)) % q for t in range(blocks * 256)]
    assert host(sink).tolist() == want
