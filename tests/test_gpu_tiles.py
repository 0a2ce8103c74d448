"""The walk of the eight-wavefront tiles over their 32-token blocks, where it can go wrong: one block, a remainder of
its unrolled steps, a last block with few tokens (slots behind them read as NaN), a causal edge inside any of the last
blocks, wavefronts whose rows are all padding; whole tiles, and tiles cut into key chunks, whose walk begins at a later block
and ends before the tile's last."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.driver import run_workload as run_oracle
from paper_2510_25412_amd import driver, synth

pytestmark = pytest.mark.gpu

LENS = [0, 1, 15, 31, 32, 33, 63, 64, 95, 97, 127, 128, 161, 200, 255, 290]
NEW = [16, 17, 31, 32, 33, 47, 64, 65, 100, 129]


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (16, 8), (32, 8), (16, 2)])
@pytest.mark.parametrize("lips", [2, 40])
def test_tiles_of_every_number_of_blocks(Hq, Hkv, lips):
    files = [LENS[(5 * i + lips) % len(LENS)] for i in range(lips)]
    new = [NEW[(3 * i + Hq) % len(NEW)] for i in range(lips)]
    shape = synth.Shape(Hq, Hkv, 128, 16, synth.BF16)
    pages = sum(-(-(n + m) // 16) + 1 for n, m in zip(files, new)) + 8
    wl = synth.custom(f"tiles{Hq}_{Hkv}_{lips}", shape, [("new", n) for n in files], list(enumerate(new)), pages, seed=70 + Hq + lips)
    print(f"[case] {wl.name}", flush=True)
    got, sess = driver.run_workload(wl, poison=True)
    ref, _ = run_oracle(wl, dtype=np.float64)
    assert np.isfinite(got).all()
    # weights are rounded to 11 bits: half a unit, 2^-12 of a weighted mean of |v| <= 5 or so
    assert float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max()) <= 2e-3
    sess.close()


# files of one batch and their new tokens: ends at many offsets in a block, pieces of every remainder of the steps unrolled by four,
# pieces that begin inside the tile's own tokens (some of its rows see none of their keys)
CUT = [([2500], [16]), ([3001], [33]), ([4000], [100]), ([5017], [65]), ([6100], [47]), ([7990], [129]), ([9000], [17]), ([1203], [257]),
       ([0], [700]), ([130], [900]), ([1800, 2600], [64, 31]), ([4000, 17, 1203], [16, 700, 33])]


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (16, 8), (32, 8), (16, 2)])
def test_key_chunks_of_every_number_of_blocks(Hq, Hkv):
    shape, tokens = synth.Shape(Hq, Hkv, 128, 16, synth.BF16), 256 * Hkv // Hq
    for files, new in CUT:
        pages = sum(-(-(n + m) // 16) + 1 for n, m in zip(files, new)) + 8
        wl = synth.custom(f"chunks{Hq}_{Hkv}_{files[0]}_{new[0]}", shape, [("new", n) for n in files], list(enumerate(new)), pages, seed=90 + Hq + files[0])
        print(f"[case] {wl.name}", flush=True)
        got, sess = driver.run_workload(wl, poison=True)
        assert sess.ctx.get_stats()["last_batch_tiles"] > sum(-(-n // tokens) for n in new) * Hkv      # cut
        ref, _ = run_oracle(wl, dtype=np.float64)
        assert np.isfinite(got).all()
        assert float((np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max()) <= 2e-3          # as above
        sess.close()
