"""lumen_kv_ckpt_status reads and clears the error word of its own workspace,
also from more host threads at once than the library has words to receive
codes in, each on a stream of its own."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2606_17787_amd.kvckpt as kv
from paper_2606_17787_amd.workloads import CacheShape, NHD

from gpu_util import dev, h2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [1, 80])
def test_every_thread_reads_its_own_word(threads):
    out, errors = [None] * threads, []
    start = threading.Barrier(threads)

    def work(i):
        try:
            s = torch.cuda.Stream()
            # odd threads plan an invalid range (RANGE), even ones a good one
            b = h2d(np.array([4], np.int32))
            e = h2d(np.array([3 if i % 2 else 9], np.int32))
            ws = kv.new_workspace(1, dev())
            torch.cuda.synchronize()
            start.wait(60)
            got = []
            for _ in range(5):
                kv.lumen_kv_ckpt_plan(b, e, ws, stream=s)
                got.append(kv.lumen_kv_ckpt_status(ws, stream=s))
                got.append(kv.lumen_kv_ckpt_status(ws, stream=s))  # cleared
            out[i] = got
        except BaseException as x:  # reported by the main thread
            errors.append(x)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(100)
    assert not errors, errors[0]
    for i in range(threads):
        bad = kv.LUMEN_ERR_RANGE if i % 2 else kv.LUMEN_OK
        assert out[i] == [bad, kv.LUMEN_OK] * 5


@pytest.mark.parametrize("handle", [0, 1, 2],
                         ids=["null", "hipStreamLegacy", "hipStreamPerThread"])
def test_streams_that_are_names(handle):
    """Every entry point that takes a stream takes the runtime's named ones:
    a plan, a pack over it and the status, on the handle itself."""
    lib = kv.load_library()
    shape = CacheShape(2, 2, 16, 4, NHD)
    nb = 3
    lay = kv.layout(shape, nb)
    src = torch.arange(shape.pool_elems(nb), dtype=torch.int16, device=dev())
    ck = torch.zeros(4 * shape.token_row_elems, dtype=torch.int16,
                     device=dev())
    bt = h2d(np.array([[2], [1]], np.int32))
    s, e = h2d(np.array([0, 0], np.int32)), h2d(np.array([4, -1], np.int32))
    ws = kv.new_workspace(2, dev())
    torch.cuda.synchronize()
    assert lib.lumen_kv_ckpt_plan(s.data_ptr(), e.data_ptr(), 2, 0, None,
                                  ws.data_ptr(), handle) == 0
    assert lib.lumen_kv_ckpt_pack(ctypes.byref(lay), src.data_ptr(),
                                  bt.data_ptr(), 1, 2, ws.data_ptr(),
                                  ck.data_ptr(), 4, handle) == 0
    assert lib.lumen_kv_ckpt_status(ws.data_ptr(), handle) == \
        kv.LUMEN_ERR_RANGE
    assert lib.lumen_kv_ckpt_status(ws.data_ptr(), handle) == kv.LUMEN_OK
    block = src.view(shape.num_layers, 2, nb, 4, -1)[:, :, 2]
    assert torch.equal(ck.view(4, shape.num_layers, 2, -1),
                       block.permute(2, 0, 1, 3))
