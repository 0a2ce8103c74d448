"""Appends whose slot map comes with the kernel's arguments (few runs of consecutive slots) and appends whose map is
read from pinned memory, on both sides of the line and at the edges of pages: every row reads back bit for bit, the
attention kernel's own appends (single tokens) beside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_25412_amd import driver, synth

pytestmark = pytest.mark.gpu


# 128 runs are the most that travel with the arguments: 2041 tokens from slot 7 on are 128 runs, 2057 are 129
@pytest.mark.parametrize("before,new", [([0], [1]), ([7], [9]), ([7], [10]), ([7], [2041]), ([7], [2057]), ([0, 15, 16, 31], [1, 2, 16, 33]),
                                        ([3] * 64, [13] * 64), ([3] * 64, [14] * 64), ([3] * 64 + [9], [14] * 64 + [1]), ([40] * 70, [1, 5] * 35),
                                        # 128 whole pages, the most tokens that 128 runs hold; the workgroups' lines at five tokens each
                                        ([0], [2048]), ([0] * 32, [64] * 32), ([7], [2559]), ([7], [2560]), ([7], [3584])])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
def test_appended_rows_read_back(before, new, dtype):
    print(f"[case] runs {before[:4]} {new[:4]} x{len(new)} {dtype}", flush=True)
    D, H, tdt = (128, 8, torch.bfloat16) if dtype == synth.BF16 else (64, 3, torch.float32)
    n_pages = sum(-(-(a + b) // 16) for a, b in zip(before, new)) + 4
    sess = driver.HipSession(synth.Shape(H, H, D, 16, dtype), n_pages, max_lips=len(new), max_tokens=4096, max_entries=8192, poison=True)
    g = torch.Generator().manual_seed(len(new) + sum(new))
    rows = lambda n: torch.randn((n, H, D), generator=g).to(tdt).cuda()  # noqa: E731
    files, old = [], []
    for n in before:
        files.append(sess.ctx.kv_open(None))
        old.append((rows(n), rows(n)))
        if n:
            sess.ctx.kv_append(files[-1], n, *old[-1], sess.stream)
    T = sum(new)
    q, k, v, out = rows(T), rows(T), rows(T), torch.empty((T, H, D), dtype=torch.float32, device="cuda")
    sess.ctx.pred_batch(files, new, q, k, v, out, sess.stream)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    t = 0
    for h, n, m, (ko, vo) in zip(files, before, new, old):
        got_k, got_v = torch.empty((n + m, H, D), dtype=tdt, device="cuda"), torch.empty((n + m, H, D), dtype=tdt, device="cuda")
        sess.ctx.kv_read(h, 0, n + m, got_k, got_v, sess.stream)
        torch.cuda.synchronize()
        assert torch.equal(got_k, torch.cat([ko, k[t:t + m]])) and torch.equal(got_v, torch.cat([vo, v[t:t + m]]))
        t += m
    sess.close()
