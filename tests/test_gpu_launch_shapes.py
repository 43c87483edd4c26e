"""The sizes at which a call changes the shape of its launch, against the CPU oracle: edges of tiles, remainders, the
smallest and largest size of each variant.  Tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest

import chain
import oracle
from paper_2101_07706_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2101_07706_amd import csgs
    csgs.lib()
    return torch.device("cuda:0")


def _csr(rng, lens, n_cols):
    rowptr = np.zeros(len(lens) + 1, np.int32)
    np.cumsum(lens, out=rowptr[1:])
    return rowptr, rng.integers(0, n_cols, int(rowptr[-1])).astype(np.int32), rng.standard_normal(int(rowptr[-1])).astype(np.float32)


# F picks the lanes per row (4, 8, 16, 32, 64); the row counts lie at the ends of the ranges in which a wavefront takes
# 2, 4, ..., 64 rows: 512 blocks of 4 wavefronts over all feature slices
@pytest.mark.parametrize("F,bf16,rows", [(256, False, (1, 9, 2016, 2017, 4033, 8065, 16128, 16129)), (64, False, (1, 33, 16352, 16353, 65409)),
                                         (128, False, (7, 4088, 4089, 65409)), (100, True, (3, 8176, 8177, 32705)),
                                         (75, False, (1, 2045, 4089, 16369))])
def test_aggregate_rows_per_wavefront(dev, F, bf16, rows):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(31 * F)
    n_cols = 3000
    X = rng.standard_normal((n_cols, F)).astype(np.float32)
    Xh = synth.to_bf16_bits(X) if bf16 else X
    Xd = torch.from_numpy(Xh.view(np.int16) if bf16 else Xh).to(dev)
    for n in rows:
        print(f"[aggregate] {n} rows, F={F} bf16={bf16}", flush=True)
        lens = rng.poisson(2, n)
        lens[rng.integers(0, n, 4)] = (0, 300, 257, 90)       # the block-wide path, and rows longer than a share
        rowptr, col, val = _csr(rng, lens, n_cols)
        want = oracle.aggregate(rowptr, col, val, Xh, relu_on_input=True)
        Z = torch.full((n + 3, F), float("nan"), dtype=torch.float32, device=dev)
        t = lambda a: torch.from_numpy(a).to(dev)
        csgs.csgs_aggregate(t(rowptr), t(col), t(val), None, Xd, None, None, True, Z[:n])
        torch.cuda.synchronize()
        chain.assert_close(Z[:n].cpu().numpy(), want, chain.RTOL, chain.ATOL, f"aggregate {n} rows F={F}")
        assert bool(torch.isnan(Z[n:]).all()), f"{n} rows: wrote past the last row"
