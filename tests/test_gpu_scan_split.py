"""The scan's work split where its group count changes: pages around multiples of the smallest group, one sequence
and many, empty ones between, head counts below and above one work-group's eight waves."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import assert_rows_close, dev, gpu_cache, oracle_pool

pytestmark = pytest.mark.gpu

CASES = [
    ([1], 8, 8), ([16 * 8], 4, 1), ([16 * 8 + 1], 1, 1), ([16 * 29], 32, 8), ([16 * 32 + 5], 8, 2),
    ([1] * 9, 4, 1), ([0, 3, 0, 640, 17, 0], 8, 2), ([16] * 20 + [300], 4, 4), ([64, 65, 63, 1, 0, 129, 40, 31], 8, 1),
    ([5, 700], 20, 10), ([2100], 4, 1),
    # up to 256 sequences a thread of the split serves a group, beyond it serves sequences
    ([16, 0, 1, 40] * 64, 4, 1), ([5, 0, 33] * 100, 4, 1),
]


@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("max_ctx", ["exact", "loose"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{len(c[0])}x{max(c[0])}-{c[1]}x{c[2]}")
def test_split_over_groups(case, max_ctx, G):
    lens, Hq, H = case
    w = W.make_workload(1, batch=len(lens), ctx_lens=np.array(lens), num_q_heads=Hq, num_kv_heads=H, d_model=None)
    pool = oracle_pool(w, group=G)
    cache = gpu_cache(pool)
    # a caller may bound the lengths tightly or by the model's maximum: the host's plan and the groups
    # the device then uses differ, the result does not
    bound = max(lens) if max_ctx == "exact" else 16 * 1024
    out = K.int2kv_decode(cache, dev(w.q), dev(w.block_table), dev(w.ctx_lens), bound, dev(w.R_k), dev(w.R_v))
    torch.cuda.synchronize()
    ref = O.decode(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v)
    assert_rows_close(out.cpu().numpy(), ref, what=str(case))
