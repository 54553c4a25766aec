"""pg_status_check through the pinned words that the device writes: several
threads on streams of their own read back their own words, an overflow reports
the count, a failed sort raises, and a call during capture is still refused."""
import threading

import pytest
import torch

import synth
from paper_2602_23040_amd import _abi as abi
from parity import renderer

pytestmark = pytest.mark.gpu


def test_status_words_of_threads_and_streams():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[gpu] status words", flush=True)
    r = renderer(synth.random_scene(side=4))        # a view table: the words exist
    dev = "cuda:0"
    bad = []

    def work(k):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            over = torch.zeros(1, dtype=torch.int32, device=dev)
            n = torch.zeros(2, dtype=torch.int64, device=dev)
            for i in range(60):
                want = (1 << 33) + 1000 * k + i
                n[0] = want
                over[0] = i % 2
                got = abi.pg_status_check(over, n)
                if got != (bool(i % 2), want):
                    bad.append((k, i, got))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    over, n = torch.full((1,), 2, dtype=torch.int32, device=dev), torch.zeros(2, dtype=torch.int64, device=dev)
    with pytest.raises(abi.PGError):
        abi.pg_status_check(over, n)
    over.zero_()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        n.add_(1)
        with pytest.raises(abi.PGError):
            abi.pg_status_check(over, n)
    g.replay()
    assert abi.pg_status_check(over, n) == (False, 1)
    r.close()
