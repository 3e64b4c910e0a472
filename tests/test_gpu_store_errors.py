"""GPU tests of epd_store_hash beside errors that are not its own: an error that the program left
uncollected, and a stream that is being captured."""

import ctypes as C

import numpy as np
import pytest
import torch

from oracle import mm_store as S
from paper_2601_11590_amd import binding as B

pytestmark = pytest.mark.gpu


def data(seed):
    rng = np.random.default_rng(seed)
    lens = [int(v) for v in rng.integers(1, 100000, size=3)]
    host = rng.integers(0, 256, size=sum(lens), dtype=np.uint8)
    off = np.concatenate([[0], np.cumsum(lens)])
    keys = [S.hash128(host[off[i]:off[i + 1]].tobytes(), i) for i in range(3)]
    return torch.from_numpy(host).to("cuda:0"), off, keys


def right(store, d):
    got = store.hash(d[0], d[1], [0, 1, 2])
    assert [(int(a), int(b)) for a, b in got] == d[2]


def test_keys_beside_an_uncollected_error():
    hip = C.CDLL("libamdhip64.so.7")
    store = B.MMStore(2 << 20)
    sets = [data(i) for i in range(4)]
    torch.cuda.synchronize()
    for d in sets:
        assert hip.hipSetDevice(4096) != 0           # refused; the error waits to be collected
        right(store, d)
    hip.hipGetLastError()
    for d in sets:
        right(store, d)
    store.close()


def test_a_capturing_stream_is_refused_and_stays_usable():
    store = B.MMStore(2 << 20)
    sets = [data(i) for i in range(3)]
    right(store, sets[0])
    x = torch.zeros(256, device="cuda:0")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        x.add_(1.0)
        with pytest.raises(B.StoreError) as e:
            store.hash(sets[1][0], sets[1][1], [0, 1, 2])
        x.add_(1.0)
    assert e.value.status == B.EPD_ERR_HIP
    for i in range(3):
        g.replay()
        right(store, sets[i])
        torch.cuda.synchronize()
        assert float(x.min()) == float(x.max()) == 2.0 * (i + 1)
    store.close()
