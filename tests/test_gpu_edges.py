"""GPU parity at the edges of the kernels' dispatch rules and tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import twilight_oracle as O
from workloads import synth
from tests.gpu_util import u16

pytestmark = pytest.mark.gpu


def _T():
    import paper_2502_02770_amd as T
    return T


@pytest.mark.parametrize("P", [1, 2, 64, 256, 257, 512, 513, 2048, 2049, 8192, 8193, 32768, 32769])
def test_page_lists_at_the_row_lengths_of_the_selection_kernels(P):
    """Random page bounds, rows one entry short of, at and beyond the length where the next selection kernel takes
    over, budgets of one page, half of the row and all but one page: page lists bit for bit."""
    T = _T()
    rng = np.random.default_rng(P)
    table = torch.arange(P, dtype=torch.int32).view(1, P)
    n = 16 * P - 3 if P > 1 else 16
    cache = T.PagedKV(2, 1, table, torch.tensor([n]), P, need_v=False)
    mm = torch.from_numpy(np.sort(rng.standard_normal((P, 1, 2, 128)).astype(np.float32), axis=2)).to(torch.bfloat16)
    mm[rng.integers(0, P, size=P // 4)] = mm[0].clone()                    # some pages tie
    cache.page_minmax.copy_(mm)
    q = torch.from_numpy(rng.standard_normal((1, 2, 128)).astype(np.float32)).to(torch.bfloat16)
    for budget in sorted({16, 16 * max(1, P // 2), 16 * max(1, P - 1)}):
        st = T.DecodeStep(cache, max_sel=max(1, budget // 16))
        st.select(q.cuda(), torch.tensor([budget], dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        for h in range(2):
            U = O.page_upper_bounds(synth.bits(q[0, h]), u16(mm[:, 0, 0]), u16(mm[:, 0, 1]))
            want = O.select_pages(U, budget, n)
            assert st.sel_pages[0, h, :int(st.sel_count[0, h])].cpu().numpy().tolist() == want.tolist(), (budget, h)
