"""GPU: turns that follow each other without a wait -- batches laid out, grown, attended and released back to back, their
uploads sharing the library's pinned staging -- against the same turns with a device synchronisation after every call."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


class Session:
    """One cached context under three models, bf16, driven turn by turn."""

    def __init__(self, seed):
        from paper_2602_12029_amd import binding as B
        rng = np.random.default_rng(seed)
        self.B, self.len = B, np.array([200 + 37 * seed], np.int32)
        self.geo = B.geometry(8, 2, 128, 16, "bf16", "bf16")
        blocks = 64
        self.pool = B.ps_pool_create(blocks, rng.permutation(blocks).astype(np.int32))
        self.keep = B.ps_kv_layout(self.pool, self.geo, self.len, [0], [0], [0])
        t = B.ps_layout_tables(self.keep, 1, 1)
        self.adopt = [t["prefix_blk"][:int(self.len[0]) // 16]]
        gen = torch.Generator().manual_seed(seed)
        def draw(*shape):
            return torch.randn(*shape, generator=gen).to(torch.bfloat16).cuda()
        self.kv = draw(blocks, 2, 2, 16, 128)
        self.tail = [draw(int(self.len[0]) % 16, 2, 128) for _ in range(2)]
        self.q = [draw(3, 8, 128) for _ in range(20)]
        self.new = [(draw(3, 2, 128), draw(3, 2, 128)) for _ in range(20)]
        torch.cuda.synchronize()

    def turn(self, steps, wait):
        from paper_2602_12029_amd.runtime import DecodeBatch
        B = self.B
        done = torch.cuda.synchronize if wait else (lambda: None)
        layout = B.ps_kv_layout_adopt(self.pool, self.geo, self.len, self.adopt, [0, 0, 0], [0, 1, 2], [0, 0, 0])
        batch = DecodeBatch(layout, self.geo, 3, self.q[0], self.kv)
        batch.kv_ingest(0, *self.tail)
        outs = []
        for i in range(steps):
            batch.append_step(self.pool, *self.new[i])
            done()
            batch.q = self.q[i]
            batch.decode_attention()
            done()
            outs.append(batch.out.clone())
        B.ps_layout_release(self.pool, layout)
        return outs

    def turns(self, wait):
        return [o for steps in (1, 5, 18, 2, 2, 20) for o in self.turn(steps, wait)]

    def close(self):
        torch.cuda.synchronize()
        self.B.ps_layout_release(self.pool, self.keep)
        self.B.ps_pool_destroy(self.pool)


def _same(a, b):
    return len(a) == len(b) and all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b))


def test_turns_without_waits_and_after_the_pools_are_gone():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for _ in range(2):                       # the second round starts with nothing kept
        s = Session(1)
        want = s.turns(True)
        assert _same(s.turns(False), want)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            got = s.turns(False)
        torch.cuda.synchronize()
        assert _same(got, want)
        s.close()


def test_turns_of_several_threads_on_their_own_streams():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sessions = [Session(i) for i in range(4)]
    want = [s.turns(True) for s in sessions]
    got = [None] * len(sessions)

    def work(i):
        torch.cuda.set_device(0)
        with torch.cuda.stream(torch.cuda.Stream()):
            got[i] = sessions[i].turns(False)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sessions))]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for s, g, w in zip(sessions, got, want):
        assert _same(g, w)
        s.close()


def test_append_step_is_ordered_in_front_of_other_streams():
    """A pass over the shared segments, which needs nothing of the step's own token, on another stream right behind
    append_step while the upload is still held up: it waits for the tables there, as for the host before."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    s = Session(3)
    layout = B.ps_kv_layout_adopt(s.pool, s.geo, s.len, s.adopt, [0, 0, 0], [0, 1, 2], [0, 0, 0])
    batch = DecodeBatch(layout, s.geo, 3, s.q[0], s.kv)
    batch.kv_ingest(0, *s.tail)
    side = torch.cuda.Stream()
    busy = torch.randn(4096, 4096, device="cuda")
    for i in range(4):
        torch.cuda.synchronize()
        for _ in range(20):
            torch.mm(busy, busy)                   # some milliseconds in front of the upload
        batch.append_step(s.pool, *s.new[i])
        with torch.cuda.stream(side):
            batch.prefix_attention()
            got = batch.workspace.clone()
        torch.cuda.synchronize()
        batch.prefix_attention()
        torch.cuda.synchronize()
        assert torch.equal(got, batch.workspace)   # (slots the pass does not write hold what they held)
    B.ps_layout_release(s.pool, layout)
    s.close()


def test_append_step_is_refused_under_capture():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    s = Session(4)
    layout = B.ps_kv_layout_adopt(s.pool, s.geo, s.len, s.adopt, [0, 0, 0], [0, 1, 2], [0, 0, 0])
    batch = DecodeBatch(layout, s.geo, 3, s.q[0], s.kv)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(RuntimeError):
            batch.append_step(s.pool, *s.new[0])
    assert not B.ps_layout_lengths(layout, 1, 3)["suffix_len"].any()
    batch.append_step(s.pool, *s.new[0])
    # the step's attention recorded behind it and replayed, as before
    batch.decode_attention()
    want = batch.out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        batch.decode_attention()
    for _ in range(3):
        batch.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _same([batch.out], [want])
    B.ps_layout_release(s.pool, layout)
    s.close()


def test_addresses_of_other_integer_types():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    from paper_2602_12029_amd.runtime import DecodeBatch
    s = Session(2)
    batch = DecodeBatch(s.keep, s.geo, 1, s.q[0][:1].contiguous(), s.kv)
    batch.decode_attention()
    want = batch.out.clone()
    batch.out.zero_()
    stream = torch.cuda.current_stream().cuda_stream
    B.ps_decode_attention(s.keep, np.int64(batch.tables.data_ptr()), np.uint64(batch.q.data_ptr()), batch.kv.data_ptr(), None,
                          batch.workspace.data_ptr(), batch.out.data_ptr(), np.int64(0), stream)
    assert _same([batch.out], [want])
    with pytest.raises(B.PsError):
        B.ps_decode_attention(s.keep, 0, batch.q.data_ptr(), batch.kv.data_ptr(), 0, batch.workspace.data_ptr(),
                              batch.out.data_ptr(), 0, stream)
    s.close()


@pytest.mark.parametrize("requests", [3, 250, 1100, 3000])
def test_uploads_recorded_in_a_graph(requests):
    """Replays bring the tables again after other layouts came and went; once the layout is released, the next ones upload
    as usual (its buffers are not handed on, and its events, which cannot be asked, are no error of theirs)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    geo = B.geometry(8, 8, 128, 16, "bf16", "bf16")
    pool = B.ps_pool_create(requests * 10, None)

    def new_layout(suffix):
        return B.ps_kv_layout(pool, geo, [40] * requests, np.arange(requests), np.zeros(requests, int), [suffix] * requests)

    def upload(layout):
        dev = torch.full((B.ps_layout_device_bytes(layout),), 0x5a, dtype=torch.uint8, device="cuda")
        B.ps_layout_upload(layout, dev.data_ptr(), torch.cuda.current_stream().cuda_stream)
        return dev

    def others():
        for suffix in (1, 17, 30):
            lay = new_layout(suffix)
            t = B.ps_layout_tables(lay, requests, requests)
            ids = np.concatenate([t["prefix_blk"], t["suffix_blk"]])
            for _ in range(3):
                assert np.array_equal(upload(lay).cpu().numpy().view(np.int32)[:ids.size], ids)
            B.ps_layout_release(pool, lay)

    layout = new_layout(20)
    want = [upload(layout) for _ in range(2)][0].cpu()       # both of its buffers exist
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    dev = torch.zeros_like(want, device="cuda")
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        B.ps_layout_upload(layout, dev.data_ptr(), torch.cuda.current_stream().cuda_stream)
    for _ in range(4):
        dev.fill_(0xa5)
        graph.replay()
        others()
        torch.cuda.synchronize()
        assert torch.equal(dev.cpu(), want)
    del graph
    torch.cuda.synchronize()
    B.ps_layout_release(pool, layout)
    others()
    B.ps_pool_destroy(pool)


@pytest.mark.parametrize("requests", [1, 3, 40, 250, 1100, 3000])
def test_uploaded_tables_are_the_layouts(requests):
    """Table blobs on both sides of 16 KiB and of 1 MiB arrive whole, whichever way they go up, and as they were when their
    upload was called."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_12029_amd import binding as B
    geo = B.geometry(8, 8, 128, 16, "bf16", "bf16")
    pool = B.ps_pool_create(requests * 6, None)
    layout = B.ps_kv_layout(pool, geo, [40] * requests, np.arange(requests), np.zeros(requests, int), [30] * requests)
    stream = torch.cuda.current_stream().cuda_stream
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    sent = []
    for rep in range(6):                     # more uploads than the layout has staging buffers, the tables changing in between
        if rep % 2 == 0:
            for _ in range(10):              # ... and the stream held up, so that a buffer read late would show
                torch.mm(busy, busy)
        n = B.ps_layout_device_bytes(layout)
        dev = torch.full((n + 64,), 0x5a, dtype=torch.uint8, device="cuda")
        B.ps_layout_upload(layout, dev.data_ptr(), stream)
        sent.append((n, dev, B.ps_layout_tables(layout, requests, requests)))
        B.ps_layout_append(pool, layout, requests, np.arange(requests) % (rep + 1) == 0)
    torch.cuda.synchronize()
    for n, dev, t in sent:
        words = dev[:n].cpu().numpy().view(np.int32)
        k = t["prefix_blk"].size
        assert np.array_equal(words[:k], t["prefix_blk"]) and np.array_equal(words[k:k + t["suffix_blk"].size], t["suffix_blk"])
        # the blob ends with the order the shared blocks are walked in, then the private ones as stored (and padding)
        entries = k + t["suffix_blk"].size
        tail = words[words.size - (entries + 3) // 4 * 4:][:entries]
        assert np.array_equal(np.sort(tail[:k]), np.arange(k)) and np.array_equal(tail[k:], np.arange(k, entries))
        assert (dev[n:] == 0x5a).all()
    assert sent[0][2]["suffix_blk"].size < sent[-1][2]["suffix_blk"].size
    print(requests, n)
    B.ps_layout_release(pool, layout)
    B.ps_pool_destroy(pool)
