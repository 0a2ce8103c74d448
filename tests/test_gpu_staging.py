"""Calls queued one behind the other with no wait in between, so that the ring of pinned staging buffers comes round while the GPU is
behind, and a call recorded into a graph: outputs and rows as when every call is waited for."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_25412_amd import driver, synth

pytestmark = pytest.mark.gpu

SHAPE = synth.Shape(16, 4, 128, 16, synth.BF16)


def _rows(g, *shape):
    return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)


def _session(pages, layers=1):
    return driver.HipSession(SHAPE, pages, max_lips=32, max_tokens=4096, max_entries=1 << 14, poison=True, n_layers=layers)


def _queue(layers, wait):
    """A fixed mix of batches, appends, extracts and merges on one context; outputs and the bytes of the pool."""
    sess, rng, g = _session(3000, layers), np.random.default_rng(5), torch.Generator(device="cuda").manual_seed(layers)
    ctx, keep, outs = sess.ctx, [], []
    files = [ctx.kv_open(None) for _ in range(12)]
    big = torch.zeros((8192, 8192), dtype=torch.bfloat16, device="cuda")

    def done():
        if wait:
            torch.cuda.synchronize()
        else:
            torch.mm(big, big)                    # about a millisecond: the GPU falls behind
    for f, n in zip(files, rng.integers(1, 900, 12)):
        k, v = _rows(g, layers, n, 4, 128), _rows(g, layers, n, 4, 128)
        keep += [k, v]
        ctx.kv_append(f, int(n), k, v, sess.stream)
        done()
    for step in range(160):
        live = [int(f) for f in rng.choice(files, rng.integers(1, 12), replace=False)]
        if step % 4 < 2:
            new = [int(x) for x in rng.choice([1, 1, 1, 3, 40], len(live))]
            T = sum(new)
            q, k, v, out = _rows(g, layers, T, 16, 128), _rows(g, layers, T, 4, 128), _rows(g, layers, T, 4, 128), torch.zeros((layers, T, 16, 128), device="cuda")
            keep += [q, k, v]
            outs.append(out)
            if layers == 1:
                (ctx.pred_batch if step % 8 else ctx.pred_batch_static)(live, new, q[0], k[0], v[0], out[0], sess.stream)
            else:
                ctx.pred_begin(live, new, sess.stream)
                for layer in range(layers):
                    ctx.pred_layer(layer, q[layer], k[layer], v[layer], out[layer], sess.stream)
        elif step % 4 == 2:
            n = int(rng.choice([1, 30, 2100 if step == 42 else 200]))
            k, v = _rows(g, layers, n, 4, 128), _rows(g, layers, n, 4, 128)
            keep += [k, v]
            ctx.kv_append(live[0], n, k, v, sess.stream)
        else:
            idx = [rng.permutation(ctx.kv_len(f))[:ctx.kv_len(f) // 2] for f in live[:3]]
            made = ctx.kv_extract_batch(live[:3], idx, sess.stream) + [ctx.kv_merge(live[:2], sess.stream)]
            out = torch.zeros((2, ctx.kv_len(made[0]), 4, 128), dtype=torch.bfloat16, device="cuda")
            outs.append(out)
            if out.shape[1]:
                ctx.kv_read(made[0], 0, out.shape[1], out[0], out[1], sess.stream)
            for h in made:
                ctx.kv_remove(h)
        done()
    end = torch.cuda.Event()
    end.record()
    assert wait or not end.query()                # it still is
    torch.cuda.synchronize()
    lengths = [ctx.kv_len(f) for f in files]
    result = lengths, [o.cpu() for o in outs], sess.pool.cpu()
    sess.close()
    return result


@pytest.mark.parametrize("layers", [1, 3])
def test_calls_queued_without_a_wait(layers):
    print(f"[case] queued calls, layers={layers}", flush=True)
    lengths, outs, pool = _queue(layers, wait=True)
    for repeat in range(2):
        lengths2, outs2, pool2 = _queue(layers, wait=False)
        assert lengths2 == lengths and len(outs2) == len(outs) > 100
        assert all(torch.equal(a, b) for a, b in zip(outs, outs2))
        assert torch.equal(pool, pool2)


@pytest.mark.parametrize("new", [[1, 1, 1], [1, 20, 5]])
def test_a_call_recorded_into_a_graph(new):
    print(f"[case] recorded call, new={new}", flush=True)
    sess, g = _session(600), torch.Generator(device="cuda").manual_seed(3)
    ctx, files = sess.ctx, []
    for n in (40, 333, 1000):
        k, v = _rows(g, n, 4, 128), _rows(g, n, 4, 128)
        files.append(ctx.kv_open(None))
        ctx.kv_append(files[-1], n, k, v, sess.stream)
        torch.cuda.synchronize()
    T, lengths = sum(new), [ctx.kv_len(f) for f in files]
    q, k, v = _rows(g, T, 16, 128), _rows(g, T, 4, 128), _rows(g, T, 4, 128)

    def eager():
        out = torch.zeros((T, 16, 128), device="cuda")
        ctx.pred_batch_static(files, new, q, k, v, out, sess.stream)
        ctx.kv_truncate(files, lengths)
        torch.cuda.synchronize()
        return out
    eager()
    out, graph = torch.zeros((T, 16, 128), device="cuda"), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.pred_batch_static(files, new, q, k, v, out, sess.stream)
    ctx.kv_truncate(files, lengths)
    for replay in range(3):                       # its staging buffer is the ring's next after four calls: three in between
        q.copy_(_rows(g, T, 16, 128))
        k.copy_(_rows(g, T, 4, 128))
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert torch.isfinite(got).all() and torch.equal(got, eager()), replay
    for _ in range(6):                            # and the ring goes on, the buffer of the recorded call included
        assert torch.equal(eager(), got)
    sess.close()
