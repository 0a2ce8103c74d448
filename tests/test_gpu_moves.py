"""extract / merge on the GPU where the move kernel's page walk can go wrong: kv heads that are and are not
multiples of its unrolled passes, last pages with fewer tokens, several layers, indices in any order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_25412_amd import binding, driver, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,layers,dtype", [(1, 1, synth.BF16), (2, 3, synth.BF16), (3, 1, synth.F32), (4, 1, synth.BF16),
                                              (5, 2, synth.BF16), (8, 3, synth.F32), (12, 1, synth.BF16), (16, 1, synth.BF16),
                                              (6, 2, synth.BF16), (10, 1, synth.F32)])
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


# 240 MiB written is the line with several layers, 384 MiB with one; the list of 960 pages is 65 KB; a launch moves 65535 pages at most
@pytest.mark.parametrize("Hkv,layers,tokens,ws,launches", [(16, 2, 960 * 16 - 7, 1 << 20, 2), (16, 2, 959 * 16, 1 << 20, 1), (1, 32, 960 * 16 - 15, 1 << 20, 2),
                                                           (3, 16, 640 * 16, 1 << 20, 2), (16, 1, 3072 * 16 - 1, 1 << 20, 2), (16, 1, 3071 * 16, 1 << 20, 1),
                                                           (16, 2, 960 * 16, 65296, 2), (16, 2, 960 * 16, 65292, 1),
                                                           (1, 1, 65535 * 16 + 40, 8 << 20, 3),
                                                           # the list pinned, 2048 workgroups and more: every number of loads in flight
                                                           (2, 1, 2048 * 16 - 3, 1 << 20, 1), (2, 1, 2048 * 16 + 1, 1 << 20, 1), (4, 3, 683 * 16, 1 << 20, 1),
                                                           (3, 1, 2050 * 16 - 15, 1 << 20, 1), (8, 1, 2049 * 16, 1 << 20, 1)])
def test_list_of_a_large_move_is_brought_to_the_device_once(Hkv, layers, tokens, ws, launches):
    # its layers and heads would otherwise fetch it again and again over the host link
    print(f"[case] large move Hkv={Hkv} layers={layers} tokens={tokens} ws={ws}", flush=True)
    pages = 2 * (tokens // 16 + 2)
    cfg = binding.make_config(Hkv, Hkv, 128, 16, synth.BF16, pages, device=0, decode_waves=1, n_layers=layers)
    pool = torch.full((layers * pages * binding.page_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda")
    workspace = torch.empty(ws, dtype=torch.uint8, device="cuda")
    cfg.pool, cfg.workspace, cfg.workspace_bytes = pool.data_ptr(), workspace.data_ptr(), ws
    ctx, st = binding.Context(cfg), torch.cuda.current_stream().cuda_stream
    k, v = (torch.randint(-32768, 32767, (layers, tokens + 1, Hkv, 128), dtype=torch.int16, device="cuda").view(torch.bfloat16) for _ in range(2))
    src = ctx.kv_open(None)
    ctx.kv_append(src, tokens + 1, k, v, st)
    before = ctx.get_stats()["kernel_launches"]
    idx = np.arange(1, tokens + 1)
    idx[::7] = idx[::7][::-1].copy()                      # every page has slots of other pages
    new = ctx.kv_extract_batch([src], [idx], st)[0]
    assert ctx.get_stats()["kernel_launches"] - before == launches
    at = torch.from_numpy(idx).cuda()
    for layer in range(layers):
        got_k, got_v = (torch.empty((tokens, Hkv, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        ctx.kv_read(new, 0, tokens, got_k, got_v, st, layer=layer)
        torch.cuda.synchronize()
        for got, want in ((got_k, k), (got_v, v)):
            assert torch.equal(got.view(torch.int16), want[layer, at].view(torch.int16)), layer
    ctx.close()
