"""ab_merge_info / ab_merge_info_batched: what is asked for is checked against the workspace before any memory is
taken for it, and a slice of the layers is the slice of the whole."""
import ctypes
import resource

import pytest
import torch

from paper_2405_01067_amd import binding as abt

pytestmark = pytest.mark.gpu


def vm_bytes():
    with open("/proc/self/statm") as fh:
        return int(fh.read().split()[0]) * resource.getpagesize()


def merge(L):
    g = torch.Generator(device="cuda").manual_seed(L)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    return abt.ab_merge_batched([dict(A_copies=[rnd(96 + 32 * i, 32 * (1 + i % 2))], B_copies=[rnd(32 * (1 + i % 2), 80)], tau=0.0)
                                 for i in range(L)])


def batched(ws, first, count, sweeps=None, n_sigma=None):
    return abt.load().ab_merge_info_batched(abt._ptr(ws), first, count, sweeps, n_sigma, abt._stream())


def test_a_slice_is_the_slice_of_the_whole():
    outs = merge(5)
    ws = outs[0]["workspace"]
    whole, part = (ctypes.c_int32 * 5)(), (ctypes.c_int32 * 2)()
    values = (ctypes.c_int32 * 5)()
    assert batched(ws, 0, 5, whole, values) == 0 and list(values) == [32, 64, 32, 64, 32]
    assert list(whole) == [o["sweeps"] for o in outs]
    assert batched(ws, 3, 2, part) == 0 and list(part) == list(whole)[3:]
    assert abt.merge_info(ws, 3) == (whole[3], 64)


def test_layers_that_are_not_there_cost_no_memory():
    ws = merge(2)[0]["workspace"]
    soft, hard = resource.getrlimit(resource.RLIMIT_AS)
    resource.setrlimit(resource.RLIMIT_AS, (vm_bytes() + (1 << 30), hard))      # a table of 10^9 layers is 16 GB
    try:
        codes = [abt.load().ab_merge_info(abt._ptr(ws), 10 ** 9, None, None, abt._stream()), batched(ws, 0, 10 ** 9),
                 batched(ws, 2 ** 31 - 1, 2 ** 31 - 1), batched(ws, 1, 2), batched(ws, 2, 1)]
    finally:
        resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
    assert codes == [-1] * 5                            # ABT_EINVAL
    assert batched(ws, 1, 1) == 0
