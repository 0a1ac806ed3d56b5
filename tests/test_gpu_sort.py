"""The segmented sort against numpy's lexsort at the sizes where its paths meet: two segments to a
wavefront (up to 32 keys), one (64), block-ranked (512), bitonic in LDS (2,048), the tiles of the
offset scan (4,096 segments) and of the counting passes (1,024 keys).  Results are integers: exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(sizes, seed, rng_pos=50):
    from paper_2603_25068_amd import workloads as W
    from paper_2603_25068_amd.sim import Simulator
    rng = np.random.default_rng(seed)
    seg = rng.permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    n = len(seg)
    pos = rng.integers(-rng_pos, rng_pos, n).astype(np.float32)          # many ties, both signs, zeros
    pos[rng.random(n) < 0.05] = -0.0
    pos[rng.random(n) < 0.02] = np.inf
    seq = rng.integers(-3, 3, n).astype(np.int32)                        # equal sequences go by index
    t = lambda a: torch.from_numpy(a).cuda()
    s = Simulator(W.line())
    perm, off = s.segsort(t(seg), t(pos), t(seq), len(sizes))
    perm2, off2 = torch.empty_like(perm), torch.empty_like(off)
    s.segsort_noalloc(t(seg), t(pos), t(seq), len(sizes), perm2, off2)
    want = np.lexsort((np.arange(n), seq, -pos, seg))
    assert np.array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(sizes)]))
    assert np.array_equal(perm.cpu().numpy(), want)
    assert torch.equal(perm, perm2) and torch.equal(off, off2)


@pytest.mark.parametrize("sizes", [
    [1], [0, 0, 3], [32, 32], [33, 31], [64, 1, 65, 0, 2], [63, 64, 65, 66, 67, 68, 69, 70, 71],
    [256, 257, 511, 512, 513], [1023, 1024, 1025], [2047, 2048], [0] * 7 + [2048], [5] * 4095, [3] * 4096, [2] * 4097,
])
def test_segsort_edges(sizes):
    _check(sizes, seed=len(sizes))


def test_segsort_random_segment_lengths():
    rng = np.random.default_rng(11)
    _check(rng.poisson(28, 9001), seed=12)
    _check(np.minimum(rng.geometric(0.01, 700), 2048), seed=13)


@pytest.mark.parametrize("sizes", [[2000] * 8, [2000] * 9 + [1] * 9000, [600, 100] * 20, [70] * 1100, [1] * 1025 + [65] * 9])
def test_segsort_long_segments_side_by_side(sizes):
    """Neighbouring long segments, which different workgroups take, among few and many short ones."""
    _check(sizes, seed=len(sizes))
