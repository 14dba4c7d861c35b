"""The dense operand of the matrix-core products where offsets are repeated: entries are stored until a workgroup meets an offset for
the second time and added to from then on.  Repeats within a pass of 512 diagonals, across passes, of diagonals that wrap into a
workgroup's range, and inputs that are laid out by one workgroup as a whole."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeats", ["none", "next", "pass", "many"])
@pytest.mark.parametrize("M,N,K", [(128, 128, 100), (128, 256, 250), (256, 128, 250), (768, 256, 760), (384, 1152, 1100), (1024, 1024, 1000)])
def test_repeated_offsets(M, N, K, repeats):
    D, T = max(M, N), 70
    _, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + N + K)
    rng = np.random.default_rng(K)
    offsets = rng.permutation(D)[:K].astype(np.int32)
    if repeats == "next":
        offsets[1::2] = offsets[: K // 2 * 2 : 2] - D  # the same diagonal, another number for it
    elif repeats == "pass":
        offsets[min(512, K // 2):] = offsets[: K - min(512, K // 2)]
    elif repeats == "many":
        offsets = rng.integers(-2 * D, 2 * D, K).astype(np.int32)
        offsets[K // 3: K // 2] = 5
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16")
    prepared = dd.dd_prepare(off, V, M, N)
    assert rel_err(to_host(dd.dd_fwd(x, None, None, N, prepared=prepared)), orc.fwd(X, offsets, values, N)) <= TOL["bf16"]
    assert rel_err(to_host(dd.dd_bwd_input(dy, None, None, M, prepared=prepared)), orc.bwd_input(dY, offsets, values, M)) <= TOL["bf16"]
