"""extract / merge on the GPU where the move kernel's page walk can go wrong: kv heads that are and are not
multiples of its unrolled passes, last pages with fewer tokens, several layers, indices in any order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_25412_amd import driver, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,layers,dtype", [(1, 1, synth.BF16), (2, 3, synth.BF16), (3, 1, synth.F32), (4, 1, synth.BF16),
                                              (5, 2, synth.BF16), (8, 3, synth.F32), (12, 1, synth.BF16), (16, 1, synth.BF16)])
def test_moved_rows_are_the_source_rows(Hkv, layers, dtype):
    print(f"[case] moves Hkv={Hkv} layers={layers} {dtype}", flush=True)
    D, tdt = (128, torch.bfloat16) if dtype == synth.BF16 else (64, torch.float32)
    sess = driver.HipSession(synth.Shape(Hkv, Hkv, D, 16, dtype), 96, max_lips=8, max_tokens=512, max_entries=4096, poison=True, n_layers=layers)
    g = torch.Generator().manual_seed(100 * Hkv + layers)
    rng = np.random.default_rng(Hkv)
    files, rows = [], []
    for n in (1, 45, 300):
        k, v = (torch.randn((layers, n, Hkv, D), generator=g).to(tdt).cuda() for _ in range(2))
        files.append(sess.ctx.kv_open(None))
        sess.ctx.kv_append(files[-1], n, k, v, sess.stream)
        torch.cuda.synchronize()
        rows.append((k, v))
    lists = [[0, 0, 0], rng.permutation(45)[:17], np.flatnonzero(rng.random(300) < 0.5)]
    new = sess.ctx.kv_extract_batch(files, lists, sess.stream)
    want = [tuple(x[:, np.asarray(i)] for x in r) for r, i in zip(rows, lists)]
    new.append(sess.ctx.kv_merge([files[1], files[0], files[2]], sess.stream))
    want.append(tuple(torch.cat([rows[1][x], rows[0][x], rows[2][x]], 1) for x in range(2)))
    for h, (k, v) in zip(files + new, rows + want):
        for layer in range(layers):
            got_k, got_v = torch.empty_like(k[layer]), torch.empty_like(v[layer])
            sess.ctx.kv_read(h, 0, k.shape[1], got_k, got_v, sess.stream, layer=layer)
            torch.cuda.synchronize()
            assert torch.equal(got_k, k[layer]) and torch.equal(got_v, v[layer]), (h, layer)
    sess.close()
