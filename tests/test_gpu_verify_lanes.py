"""Sums of the self-checking execute across lanes and wavefronts: a word changed anywhere in a chunk, whichever lane
and wavefront holds it, shows in all three digests; equal buffers give 0."""
import numpy as np
import pytest

from paper_1705_01598_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("n", [16384, 16384 + 1000, 3 * 16384 + 3])
def test_one_word_changed_in_any_lane(n, elem):
    rng = np.random.default_rng(n + elem)
    a = torch.from_numpy(rng.integers(-2**31, 2**31, n * elem // 4, dtype=np.int64).astype(np.int32)).cuda()
    b = a.clone()
    verdict = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    ws = torch.empty(B.verify_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream

    def compare():
        verdict.fill_(-1)
        B.tperm_multiset_compare(a.data_ptr(), b.data_ptr(), n, elem, verdict.data_ptr(), ws.data_ptr(), ws.numel(), stream)
        return int(verdict.item())

    assert compare() == 0
    words = 16 // elem                        # of one load: word i lies in lane i / words % 64 of wavefront i / words / 64 % 16
    at = {lane * words for lane in range(0, 64, 1)} | {wave * 64 * words + 37 * words for wave in range(16)} | {n - 1, n - 2, n // 2}
    for i in sorted(at):
        word = i * elem // 4
        b[word] ^= 0x10
        assert compare() == 7, i
        b[word] ^= 0x10
    assert compare() == 0
