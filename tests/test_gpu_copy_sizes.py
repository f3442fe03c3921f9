"""Block copies at block sizes around the workgroup's 64 KiB: one 16-byte chunk,
less than one chunk per thread, a whole pass, one chunk more and less, two
passes and a remainder. Exact, with skipped pairs among the others."""
import pytest
import torch

import paper_2608_23658_amd.kvattn as K
from tests.gpu_helpers import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("chunks", [1, 1000, 1025, 4095, 4096, 4097, 9300])
def test_copy_block_sizes(chunks):
    nb, L = 12, 3
    g = torch.Generator().manual_seed(401 + chunks)
    layers = [torch.randint(-2**31, 2**31 - 1, (nb, chunks * 4), generator=g, dtype=torch.int32)
              for _ in range(L)]
    src, dst = [0, 3, 7, 5, -1, 2], [1, 4, 8, 5, 9, nb]      # the last three are skipped
    want = [x.clone() for x in layers]
    for x, y in zip(want, layers):
        x[[1, 4, 8]] = y[[0, 3, 7]]
    dev = [x.cuda() for x in layers]
    say("copy blocks of", chunks * 16, "bytes")
    K.copy_blocks(dev, nb, chunks * 16, torch.tensor(src, dtype=torch.int32, device="cuda"),
                  torch.tensor(dst, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    for x, y in zip(dev, want):
        assert torch.equal(x.cpu(), y)
