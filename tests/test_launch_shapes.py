"""The default launch shape, as far as it can be seen without a GPU."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2311_12973_amd as G
from paper_2311_12973_amd import workloads as W


@pytest.mark.skipif(torch.cuda.is_available(), reason="with a device the call would go on to its stand-in addresses")
@pytest.mark.parametrize("preset,prec,score,nx,T,fits", [
    ("seir", G.PREC_FP32, True, 2150, 100, True), ("seir", G.PREC_FP32, True, 2176, 100, True),
    ("seir", G.PREC_FP32, True, 2300, 100, False), ("sir_fp64", G.PREC_FP32, True, 3329, 700, True),
    ("sir_fp64", G.PREC_FP64, True, 3265, 500, False), ("seir", G.PREC_FP64, False, 4096, 1024, True),
    ("age_seir", G.PREC_FP32, False, 2048, 1024, True), ("age_seir", G.PREC_FP64, False, 2048, 1024, True)])
def test_a_shape_is_accepted_whatever_the_number_of_filters(preset, prec, score, nx, T, fits):
    """A filter that fits in LDS in some workgroup size is accepted for every number of filters
    (the call then fails for want of a device), one that fits in none is refused for every."""
    L = G.lib()
    fake = ctypes.c_void_p(1 << 20)
    w = W.preset(preset)
    y = np.ones((T, 4 if preset == "age_seir" else 1), dtype=np.int32)
    runs = G.make_runs([dict(T=T, nx=nx, seed=1, y=y)])
    c = G.make_config(w, precision=prec)
    ws = L.smc2_pf_workspace_bytes(ctypes.byref(c), runs)
    for n in (1, 2, 100, 256, 257, 512, 513, 700, 2000, 20000):
        rc = (L.smc2_pf_score(ctypes.byref(c), n, fake, runs, 1, fake, fake, fake, ws, None) if score else
              L.smc2_pf_loglik(ctypes.byref(c), n, fake, runs, 1, fake, fake, ws, None))
        assert rc == (G.E_DEVICE if fits else G.E_ARG), (n, L.smc2_last_error(None))
