"""The sizes at which a call changes its plan or kernel, against the oracle (bars as in gpuutil)."""
import pytest
import torch

import test_gpu_parity as parity
from paper_2606_13097_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    yield


@pytest.mark.parametrize("n_seqs,n_segs,page,alias", [(1, 32, 0, False), (1, 33, 0, False), (1, 32, 16, True),
                                                      (65, 1, 16, True), (130, 1, 16, False)])
def test_graft_plan_by_value_and_uploaded(n_seqs, n_segs, page, alias):
    """Up to 32 segments of a graft go by value, more through the staging ring; page rows of up to
    64 sequences go up in one launch, more in several."""
    lengths = [1 + (37 * i) % 131 for i in range(max(n_segs, 5))]
    segs = [[(s + j) % len(lengths) for j in range(n_segs)] for s in range(n_seqs)]
    w = synth.custom(synth.Shape(2, 8, 2, 64, 1e4, "bf16"), 3, lengths, segs, 5, 1, page_size=page)
    parity.run_pipeline(w, [1], 1, [0, n_seqs - 1], alias=alias)
