"""The radix sort at the sizes where its passes change: one block and one more,
one scan tile and more, 4 keys per thread up to 2^18 and 16 beyond.  Keys,
stable permutation and leaf ranges bit for bit against the oracle's tree."""
import numpy as np
import pytest

import workloads as W
from oracle import tree as T

pytestmark = pytest.mark.gpu
L = 2 * np.pi


@pytest.mark.parametrize("n,level", [(1, 1), (1023, 2), (1025, 2), (4097, 3), (65537, 4), (1 << 18, 3),
                                     ((1 << 18) + 1, 3)])
def test_sort_is_stable_at_every_size(n, level):
    import torch
    import paper_1110_2921_amd as vm
    ctx = vm.FMM()
    x, a = W.random_particles(n, 9 + n % 97)
    dev = [torch.from_numpy(np.ascontiguousarray(v.T)).cuda() for v in (x, a)]
    print(f"[tree] n={n} level={level}", flush=True)
    ctx.gauss_sum(dev[0], dev[1], 1e-3, level, periodic=1)
    keys, perm, start = ctx.debug_tree(n, level)
    ref = T.build(x, (0, 0, 0), L, level, 1)
    assert np.array_equal(perm, ref["perm"])
    assert np.array_equal(keys, ref["keys"][ref["perm"]])
    assert np.array_equal(start, np.append(ref["start"], n))
