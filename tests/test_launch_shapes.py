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


def _default_block(model, prec, nx, T, n_filters, schedule=G.SCHED_AUTO, score=False, n_cu=256):
    f = G.lib()._ZN4smc216pf_default_blockEiiiiibii
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_bool, ctypes.c_int, ctypes.c_int]
    return f(model, prec, nx, T, schedule, score, n_filters, n_cu)


@pytest.mark.parametrize("model,prec,score,n,nx,T,fastest", [
    # rounds of wide workgroups against one of narrower ones: the rest of a day counts each round
    (G.LINGAUSS, G.PREC_FP64, False, 600, 1000, 200, 256), (G.LINGAUSS, G.PREC_FP64, False, 1200, 1000, 200, 256),
    (G.LINGAUSS, G.PREC_FP64, False, 2500, 512, 200, 256), (G.LINGAUSS, G.PREC_FP64, True, 3500, 512, 200, 256),
    (G.SEIR, G.PREC_FP32, False, 700, 1000, 60, 256), (G.SIR, G.PREC_FP64, False, 513, 1024, 60, 256),
    # a workgroup more per CU by the bytes of LDS than by its granules
    (G.SEIR, G.PREC_FP32, False, 2500, 400, 60, 256), (G.SIR, G.PREC_FP64, False, 2500, 400, 60, 256),
    (G.AGE_SEIR, G.PREC_FP32, False, 1200, 640, 40, 512), (G.AGE_SEIR, G.PREC_FP32, False, 513, 640, 40, 512),
    # sizes other than the most resident waves'
    (G.SEIR, G.PREC_FP32, False, 4096, 128, 60, 64), (G.SEIR, G.PREC_FP32, False, 3000, 257, 60, 64),
    (G.SEIR, G.PREC_FP32, False, 513, 40, 60, 192), (G.SIR, G.PREC_FP32, False, 600, 100, 60, 256),
    # a single wave's draws spread only while the CU has a wave slot free
    (G.SEIR, G.PREC_FP32, True, 2048, 64, 60, 64), (G.SEIR, G.PREC_FP64, False, 2000, 64, 60, 64),
    (G.SIR, G.PREC_FP32, False, 1000, 100, 60, 256)])
def test_many_filters_take_the_size_that_measured_fastest(model, prec, score, n, nx, T, fastest):
    """Shapes where the sizes' times lie far apart (10% to 60%): the fastest of those measured."""
    assert _default_block(model, prec, nx, T, n, score=score) == fastest


@pytest.mark.parametrize("model,prec", [(G.SIR, G.PREC_FP64), (G.SEIR, G.PREC_FP32), (G.AGE_SEIR, G.PREC_FP32)])
def test_the_size_follows_the_device_s_cus(model, prec):
    """An eighth of the filters on a partition of an eighth of the CUs run on the same size; as many
    as fill the whole card do not."""
    for nx in (64, 100, 300, 700, 1000, 2000):
        for per_cu in (0.25, 1, 2, 2.25, 4, 9, 33):
            assert (_default_block(model, prec, nx, 60, int(32 * per_cu), n_cu=32) ==
                    _default_block(model, prec, nx, 60, int(256 * per_cu)))
    assert _default_block(G.SEIR, G.PREC_FP32, 1000, 60, 256, n_cu=32) < _default_block(G.SEIR, G.PREC_FP32, 1000, 60, 256)
