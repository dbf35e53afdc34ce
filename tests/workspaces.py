"""Calls in workspaces smaller than the size functions report (shared by the GPU tests)."""
import ctypes
import re

import pytest
import torch


def scratch(nbytes):
    """That many bytes with a guard behind them, which a call must leave alone."""
    whole = torch.full((nbytes + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    return whole[:nbytes], whole[nbytes:]


def least_bytes(lib, call):
    """What the message of a refusal says; call(workspace)."""
    with pytest.raises(lib.SlhcError) as e:
        call(scratch(256)[0])
    assert e.value.status == 3
    return int(re.search(r"workspace \d+ < (\d+) bytes", str(e.value)).group(1))


def by_list_kernels(lib, call):
    """call(workspace) with so little that the half-precision engine does not fit: the list kernels run."""
    return call(scratch(least_bytes(lib, call))[0])


def cross_1nn_in(lib, Xd, colour, rows, m):
    """lib.cross_1nn in a workspace that is passed."""
    N, d = Xd.shape

    def call(ws):
        idx = torch.empty(m, dtype=torch.int32, device="cuda")
        dist = torch.empty(m, dtype=torch.float32, device="cuda")
        rc = lib.load_library().slhc_cross_1nn(Xd.data_ptr(), N, d, colour.data_ptr(), rows.data_ptr() if rows is not None else None, m,
                                               idx.data_ptr(), dist.data_ptr(), ws.data_ptr(), ws.numel(),
                                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        if rc:
            raise lib.SlhcError(rc, "", lib.load_library().slhc_last_error().decode())
        return idx, dist
    return call
