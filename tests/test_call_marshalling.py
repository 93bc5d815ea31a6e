"""Argument marshalling of the library calls: the kept workspace grows exactly when a call refuses
it, errors other than a small workspace are raised without a second call, a pass's camera array
is formed once, and the stream handle is that of the current stream."""
import ctypes

import pytest
import torch

from paper_2403_14244_amd import _abi as A
from tests.test_abi_cpu import _cam


@pytest.mark.parametrize("kept,need,calls", [(0, 100, ["query", 100]), (100, 100, [100]), (500, 100, [500]),
                                             (99, 100, [99, "query", 100]), (0, 0, ["query", 1])])
def test_workspace_grows_only_when_refused(kept, need, calls):
    seen = []

    def fn(tag, ws, size, stream):
        assert tag == "arg" and stream == 7
        n = ctypes.cast(size, ctypes.POINTER(ctypes.c_size_t))
        if not ws:
            n[0] = need
            seen.append("query")
            return A.ISOGS_OK
        seen.append(n[0])
        return A.ISOGS_OK if n[0] >= need else A.ISOGS_ERR_WORKSPACE

    ws = torch.empty(kept, dtype=torch.uint8)
    out = A.call_with_workspace(fn, ("arg",), ws, 7)
    assert seen == calls and out.numel() >= need and (out is ws) == (kept > 0 and kept >= need)


def test_other_errors_are_raised_at_once():
    seen = []

    def fn(ws, size, stream):
        seen.append(ws)
        return A.ISOGS_ERR_INVALID

    with pytest.raises(A.IsoGSError):
        A.call_with_workspace(fn, (), torch.empty(64, dtype=torch.uint8), 0)
    assert len(seen) == 1


def test_camera_batch_is_the_cameras_and_their_array():
    cams = [_cam(64, 48), _cam(33, 17)]
    batch = A.CameraBatch(cams)
    assert list(batch) == cams and A.camera_array(batch) is batch.array
    assert bytes(batch.array) == bytes(A.camera_array(cams))


@pytest.mark.gpu
def test_stream_handle_follows_the_current_stream():
    from paper_2403_14244_amd.rasterizer import _stream
    side = torch.cuda.Stream()
    for s in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(s):
            assert _stream() == torch.cuda.current_stream().cuda_stream == s.cuda_stream
