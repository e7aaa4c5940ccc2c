"""Which calls of hawkes_loglik_grad_noalloc with the dense kernels' knobs set the fixed scratch takes, read off
the status on a host without a GPU: an accepted call gets as far as asking for a device (status 3), a refused one returns
the workspace status (2).  All pointers are stand-ins and never dereferenced."""
import ctypes

import pytest
import torch

import paper_2604_01342_amd as H

FAKE = ctypes.c_void_p(4096)


def status(n, M, K=1, chunk_log2=0, **tuning):
    try:
        H.set_tuning(**tuning)
        p = H._Problem(n, M, K, 0, chunk_log2, 1.0)
        return H.lib().hawkes_loglik_grad_noalloc(ctypes.byref(p), *[FAKE] * 10, ctypes.c_void_p(0))
    finally:
        H.set_tuning()


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="stand-in pointers: only where no GPU is visible")
@pytest.mark.parametrize("call", [
    dict(n=1_000_000, M=100, dense_ranges=4),                                     # longer blocks
    dict(n=1_000_000, M=200, dense_ranges=4),
    dict(n=12_217_813, M=73, dense_ranges=16),
    dict(n=2_880_953, M=201, dense_ranges=4, dense_cols=64, dense_rows=32),
    dict(n=10_978, M=886, dense_ranges=64, dense_rows=32),                        # fewer ranges
    dict(n=260, M=896, K=3, dense_ranges=32),
    dict(n=174_233, M=1128, chunk_log2=14, dense_ranges=16, dense_cols=256),
    dict(n=309_161, M=974, dense_ranges=1, dense_rows=16),                        # shorter chunks
    dict(n=827_577, M=326, dense_ranges=2, dense_cols=128, dense_rows=32),
    dict(n=10_831_335, M=1014, chunk_log2=18, dense_cols=64),
    dict(n=16_733, M=1972, chunk_log2=16, dense_ranges=1, dense_rows=16),
])
def test_accepted(call):
    assert status(**call) == 3


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="stand-in pointers: only where no GPU is visible")
def test_refused():
    assert status(3_000_000, 1000) == 2          # nothing set: the library's own layout or none
    assert status(3_000_000, 1000, dense_ranges=4) == 2
