"""The function that gives smat_preprocess_on_device its scratch memory: what is raised in it reaches the caller, and without memory the handle is the host's.
Host code alone: the device's part of torch is replaced."""
import contextlib

import numpy as np
import pytest
import torch

import paper_2408_11551_amd as S


class Stop(BaseException):
    """As KeyboardInterrupt: not an Exception."""


def _graph(M=30000, per_row=14):
    """Rows of random columns: most are clusters of their own, and looking for partners on the device pays with any number of threads."""
    rng = np.random.default_rng(3)
    keys = np.unique(np.repeat(np.arange(M), per_row) * M + rng.integers(0, M, M * per_row))
    row_ptr = np.zeros(M + 1, np.int64)
    np.cumsum(np.bincount(keys // M, minlength=M), out=row_ptr[1:])
    return M, M, row_ptr, (keys % M).astype(np.int32), np.ones(keys.size, np.uint16), "f16"


def _device_of_torch(monkeypatch, asked, capturing, empty):
    def device(_):
        asked.append(1)
        return contextlib.nullcontext()
    monkeypatch.setattr(torch.cuda, "device", device)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
    monkeypatch.setattr(torch, "empty", empty)


def _raises(error):
    def empty(*_, **__):
        raise error
    return empty


@pytest.mark.parametrize("error", [RuntimeError("HIP error"), Stop("interrupted"), ValueError("device")])
def test_what_is_raised_reaches_the_caller(monkeypatch, capfd, error):
    asked = []
    _device_of_torch(monkeypatch, asked, False, _raises(error))
    with pytest.raises(type(error)) as caught:
        S.smat_preprocess_on_device(*_graph(), device="cuda:0")
    assert caught.value is error and asked == [1]
    assert "Exception ignored" not in capfd.readouterr().err


@pytest.mark.parametrize("capturing", [False, True])
def test_without_memory_the_handle_is_the_hosts(monkeypatch, capfd, capturing):
    args, asked = _graph(), []
    alone = S.smat_preprocess(*args)
    _device_of_torch(monkeypatch, asked, capturing, _raises(torch.cuda.OutOfMemoryError("out of memory")))
    helped = S.smat_preprocess_on_device(*args, device="cuda:0")
    assert asked == [1] and "Exception ignored" not in capfd.readouterr().err
    assert np.array_equal(S.smat_export_perm(alone, args[0]), S.smat_export_perm(helped, args[0]))
    S.smat_destroy(alone)
    S.smat_destroy(helped)
