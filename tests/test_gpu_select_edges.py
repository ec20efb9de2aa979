"""TopKMask at the edges of its kernels' work units, against the oracle, exactly: mask words (32 entries, eight per
lane, 8192 per workgroup step), tensors that fill their last vector, word or chunk by one entry or miss it by one.
"""
import numpy as np
import pytest

from oracle import numerics as nm
from oracle import ties

import paper_2607_19331_amd as iso
from tests.gpu_helpers import Unit, bits_to_mask, run_fused, run_topk, say

pytestmark = pytest.mark.gpu


def _unit(rng, n, k, dtype, K=2):
    # coarse values: many entries share the threshold magnitude, so the flat-index rule decides
    ds = []
    for _ in range(K):
        v = np.round(rng.standard_normal(n) * 6.0) / 4096.0
        v[rng.random(n) < 0.3] = 0.0
        ds.append(nm.from_f64(v, dtype))
    return Unit(1, n, nm.from_f64(np.zeros(n), dtype), ds, dtype, k)


def check(units, K, dtype):
    d, bits, st, _ = run_topk(units, K, dtype, with_bits=True)
    assert st == 0
    for j, u in enumerate(units):
        for i in range(K):
            got, want = d[j * K + i], ties.topk_descriptor(u.deltas[i], u.k, dtype)
            assert (got[0], got[2], got[3], got[4]) == want, (u.n, u.k, i, got, want)
            assert got[1] == int(nm.magnitude_key(u.deltas[i], dtype).max())
            assert np.array_equal(bits_to_mask(bits[j * K + i], u.n), ties.topk_mask(u.deltas[i], u.k, dtype)), (u.n, u.k)
            tail = int(bits[j * K + i][-1]) >> (u.n % 32 or 32)
            assert tail == 0, "bits past the end are zero"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mask_word_edges(dtype):
    rng = np.random.default_rng(71)
    units = [_unit(rng, n, k, dtype) for n in (1, 7, 8, 9, 31, 32, 33, 255, 257, 8191, 8192, 8193, 24577)
             for k in {0, 1, n // 3, n}]
    say(f"mask word edges {dtype}")
    check(units, 2, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tie_cutoff_inside_chunks(dtype):
    """The quota-th threshold entry in the first, the last and a middle segment of a chunk, in a chunk that ends
    inside a vector, and beside a tensor of several chunks."""
    rng = np.random.default_rng(72)
    units = []
    for n in (511, 512, 513, 1025, 66049, 140001, 262144):
        v = np.where(rng.random(n) < 0.5, 1.0, 2.0) * np.where(rng.random(n) < 0.5, 1.0, -1.0)
        big = int((np.abs(v) == 2.0).sum())
        for k in {big + 1, big + (n - big) // 2, n - 1}:
            units.append(Unit(1, n, nm.from_f64(np.zeros(n), dtype), [nm.from_f64(v, dtype), nm.from_f64(-v[::-1], dtype)],
                              dtype, k))
    say(f"tie cutoff {dtype}")
    check(units, 2, dtype)


@pytest.mark.parametrize("copies", [1, 40])
def test_sample_of_few_and_of_many_deltas(copies):
    """iso_update FUSED TIES around the size up to which a delta is histogrammed whole (2^20), with a few deltas
    (20: each sample split over 12 workgroups) and with more than there are CUs (332: one workgroup each)."""
    rng = np.random.default_rng(73)
    units = []
    for n in (1, 9, 4097, (1 << 20) - 1, 1 << 20, (1 << 20) + 257):
        ds = [nm.from_f64(np.round(rng.standard_normal(n) * 40.0) * (rng.random(n) > 0.5) / 65536.0, "bf16") for _ in range(2)]
        units.append(Unit(1, n, nm.from_f64(rng.standard_normal(n) * 0.02, "bf16"), ds, "bf16", (n + 4) // 5))
    want = [ties.merge_unit(u.base, u.deltas, "bf16", "ties", k=u.k)["out"] for u in units]
    small = [Unit(1, 4097, u.base, u.deltas, "bf16", u.k) for u in units[2:3] for _ in range(copies * 4)]
    say(f"sample parts, {copies} copies")
    outs, _, st = run_fused(units + small, 2, "bf16", iso.MERGE_TIES)
    assert st == 0
    for u, o, w in zip(units + small, outs, want + [want[2]] * len(small)):
        assert np.array_equal(o.view(np.uint16), w.view(np.uint16)), u.n
