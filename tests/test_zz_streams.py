"""Launches on streams other than the default one.  The last file of the suite: once a process has several streams, the default one
may be served by another hardware queue than before, and other tests ask for the dies that the first queue starts at."""
import pytest

from paper_1705_09786_amd import synth

from util import compare, gpu_train, oracle_replay

pytestmark = pytest.mark.gpu

SGD = dict(kind="sgd", lr=0.05)


@pytest.mark.parametrize("tiles", [{1: 10, 2: 17}, {1: 12, 2: 17}, {1: 5, 2: 10}])
def test_long_lone_pipelines_leave_room_on_every_die(tiles):
    """Two tree pipelines of 18 .. 32 workers on streams of their own, at the same time: either has its workers dealt to all eight
    dies in turn (from whichever die the stream's queue starts at), so that both together need at most eight of any die's 32
    compute units and neither can keep the other from starting.  Each run replays as it does alone."""
    import threading
    import torch
    dims = dict(vocab=200, emb=300, hidden=150, n_class=5)
    data = synth.make_tree(24, 99, dims, max_leaves=20)
    fp = synth.init_params("tree", dims, 3)
    out = [None, None]

    def one(k, stream):
        with torch.cuda.stream(stream):
            out[k] = gpu_train("tree", dims, fp, data, 16, 10, SGD, lookup_muf=100, tiles=tiles)

    threads = [threading.Thread(target=one, args=(k, torch.cuda.Stream())) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g in out:
        xcc = g["trainer"].amp.get_worker_placement()
        assert xcc == [(xcc[0] + w) % 8 for w in range(len(xcc))], xcc
        rt = oracle_replay("tree", dims, fp, data, g["logs"], 10, SGD, lookup_muf=100)
        compare(g, rt, len(data), opt=SGD)


def test_packed_pipelines_on_any_stream():
    """A hardware queue deals workgroups to the dies from a die of its own on, and a program with several streams meets queues
    that do not start at the first.  Packed launches -- lone pipelines of few workers, replicas -- run on each of them, a replica's
    workers on one die and replicas r and r + 1 on neighbouring ones, and replay as on the default stream."""
    import torch
    rdims = dict(vocab=20, emb=32, hidden=32, n_class=5)
    rdata = synth.make_rnn(20, 3, rdims, max_len=8)
    mdims = dict(d_in=16, hidden=24, n_class=4)
    mdata = synth.make_mlp(24, 5, mdims)
    tdims = dict(vocab=97, emb=50, hidden=37, n_class=5)
    tdata = synth.make_tree(27, 27, tdims, max_leaves=8)
    mom = dict(kind="momentum", lr=0.005, momentum=0.9)
    dies = set()
    for stream in [torch.cuda.Stream() for _ in range(8)]:
        with torch.cuda.stream(stream):
            for model, dims, data, opt, kw in (("rnn", rdims, rdata, SGD, {}), ("mlp", mdims, mdata, SGD, {}),
                                               ("mlp", mdims, mdata, mom, {}),
                                               ("tree", tdims, tdata, SGD, dict(replicas=3, tiles={1: 2, 2: 3}))):
                fp = synth.init_params(model, dims, 4)
                g = gpu_train(model, dims, fp, data, 4, 3, opt, arena_bytes=1 << 28, **kw)
                a = g["trainer"].amp
                R = kw.get("replicas", 1)
                xcc, wpr = a.get_worker_placement(), a.num_workers() // R
                for r in range(R):
                    assert set(xcc[r * wpr:(r + 1) * wpr]) == {(xcc[0] + r) % 8}, xcc
                dies.add(xcc[0])
                if R == 1 and model == "rnn":
                    rt = oracle_replay(model, dims, fp, data, g["logs"], 3, opt)
                    compare(g, rt, len(data), opt=opt)
                g["trainer"].close()
    print("dies that the streams' queues start at:", sorted(dies))
