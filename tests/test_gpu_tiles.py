"""The walk of the eight-wavefront tiles over their 32-token blocks, where it can go wrong: one block, a remainder of
its unrolled steps, a last block with few tokens (slots behind them read as NaN), a causal edge inside any of the last
blocks, wavefronts whose rows are all padding; whole tiles and tiles cut into key chunks."""
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
    # 2 files: a tile's keys are cut into chunks; 40 files: whole tiles
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
