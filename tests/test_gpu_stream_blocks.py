"""Device blocks of finished streams given to later ones: objects of other
shapes and types, several at a time, on two streams and from two threads, one
abandoned in between and after a release; curves equal the oracle's exactly."""
import threading

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [("u14", (12, 40, 70)), ("u8", (9, 33, 65)), ("u16", (7, 20, 31)), ("u14", (5, 6, 7, 40)), ("u14", (14, 45, 72))]


def image(dtype, shape, seed):
    bits = {"u8": 8, "u14": 14, "u16": 16}[dtype]
    return gen.iid(shape, bits, seed=seed)


def tensor(img):
    return torch.from_numpy(img.view(np.int16) if img.dtype == np.uint16 else img).cuda()


def test_many_streams():
    import paper_1705_02045_amd as ecc
    work = [(d, image(d, s, 40 + i)) for i, (d, s) in enumerate(CASES)]
    work = [(d, x, tensor(x), oracle.curve(x, m=ecc.THRESHOLDS[d])) for d, x in work]
    torch.cuda.synchronize()
    bad = []

    def run(stream, order):
        for i in order:
            d, x, t, ref = work[i]
            st = ecc.Stream(x.shape, d, stream=stream)
            half = ecc.Stream(x.shape, d, stream=stream)  # abandoned after one chunk
            st.push(t[:3])
            half.push(t[:2])
            st.push(t[3:])
            half.abort()
            if not (st.finish() == ref).all():
                bad.append((d, x.shape))

    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(3):
        print(f"\n[gpu] streams, pass {rep}", flush=True)
        th = [threading.Thread(target=run, args=(s, o)) for s, o in zip(streams, ([0, 1, 2, 3, 4], [4, 2, 0, 3, 1]))]
        for t in th:
            t.start()
        for t in th:
            t.join()
        run(torch.cuda.default_stream(), [0, 3])
        ecc.release_workspaces()
    assert not bad
