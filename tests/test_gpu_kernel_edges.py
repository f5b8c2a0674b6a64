"""Edges of the kernels' tiles and of the rules that choose between them, each against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def w2v():
    import paper_1606_07822_amd as m
    return m


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# ------------------------------------------------------------- Huffman
# The merge gives each of up to 128 workgroups chunks of 2,048 picks of a generation: one workgroup, a chunk for
# every workgroup, and more chunks than workgroups (a generation of equal counts is as long as the vocabulary);
# codes that fill the points' staging space (32 turns on average) and exceed it.
@pytest.mark.parametrize("V,kind", [(128 * 2048, "equal"), (128 * 2048 + 1, "equal"), (300_001, "few"),
                                    (524_289, "few"), (700_000, "wide"), (60, "deep"), (256 * 3 + 62, "deep")])
def test_huffman_across_workgroups_bit_exact(w2v, V, kind):
    rng = np.random.default_rng(V)
    if kind == "equal":
        counts = np.full(V, 7)
    elif kind == "few":
        counts = rng.choice([5, 6, 11, 5000], V, p=[0.6, 0.3, 0.0999, 0.0001])
    elif kind == "wide":
        counts = np.floor(2.0 ** rng.uniform(0, 36, V)) + 1
    else:   # 60 levels from Fibonacci counts, the rest of the words at the bottom of the tree
        fib = [1 << 10, 1 << 10]
        while len(fib) < 44:
            fib.append(fib[-1] + fib[-2])
        counts = np.concatenate([np.array(fib[2:], np.int64) * max(1, V // 1024 + 1), np.ones(V - 42)])
    counts = np.sort(counts.astype(np.int64))[::-1].copy()
    t, o = w2v.build_huffman(to_dev(counts)), oracle.build_huffman(counts)
    np.testing.assert_array_equal(t.codelen.cpu().numpy(), o.codelen)
    np.testing.assert_array_equal(t.code.cpu().numpy().view(np.uint64), o.code)
    np.testing.assert_array_equal(t.point_off.cpu().numpy(), o.point_off)
    np.testing.assert_array_equal(t.points.cpu().numpy(), o.points)
    assert t.max_len == int(o.codelen.max())


@pytest.mark.parametrize("V", [66, 74, 88])
def test_huffman_too_deep_at_any_generation_is_an_error(w2v, V):
    fib = [1, 1]
    while len(fib) < V:
        fib.append(fib[-1] + fib[-2])
    with pytest.raises(w2v.W2VError) as e:
        w2v.build_huffman(to_dev(np.array(fib[::-1], np.int64)))
    assert e.value.code == w2v.W2V_E_RANGE
