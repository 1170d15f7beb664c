"""The output projection of few batch rows (16-row blocks, all of K in one launch) around its edges: batches of 1, 16, 17,
32 and 33, rows that are no multiple of 16 or 128, from one query head to pieces of K no wave count divides."""
import numpy as np
import pytest
import torch

from oracle import int2kv_oracle as O
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import assert_rows_close, dev, gpu_cache, oracle_pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["plain", "folded", "prepared", "prepared_folded"])
@pytest.mark.parametrize("B", [1, 16, 17, 32, 33])
@pytest.mark.parametrize("Hq,H,dm", [(1, 1, 8), (3, 1, 130), (8, 2, 257), (20, 4, 4100)])
def test_projection_of_few_rows(B, Hq, H, dm, fmt):
    _check(B, Hq, H, dm, fmt)


# both sides of the bounds on rows x K (at 256 CUs): blocks just over the CUs, K of 8,192 with more than 2,048 rows of W
@pytest.mark.parametrize("fmt", ["plain", "prepared"])
@pytest.mark.parametrize("B,Hq,H,dm", [(1, 40, 8, 4100), (2, 40, 8, 4100), (12, 40, 8, 4100), (13, 40, 8, 4100), (8, 64, 8, 2056),
                                       (9, 64, 8, 2056), (4, 64, 8, 2048), (5, 64, 8, 2048)])
def test_projection_by_rows_or_tiles(B, Hq, H, dm, fmt):
    _check(B, Hq, H, dm, fmt)


def _check(B, Hq, H, dm, fmt):
    w = W.make_workload(1, batch=B, ctx_lens=np.arange(B) % 3 * 7 + 1, num_q_heads=Hq, num_kv_heads=H, d_model=dm)
    pool = oracle_pool(w)
    Wo, f = dev(w.W_o), {"plain": K.INT2KV_WO_PLAIN, "folded": K.INT2KV_WO_FOLDED, "prepared": K.INT2KV_WO_PREPARED,
                         "prepared_folded": K.INT2KV_WO_PREPARED_FOLDED}[fmt]
    if fmt == "folded":
        Wo = K.int2kv_fold_wo(Wo, dev(w.R_v), Hq)
    elif fmt != "plain":
        Wo = K.int2kv_prepare_wo(Wo, dev(w.R_v) if fmt == "prepared_folded" else None, Hq, H)
    y = K.int2kv_decode(gpu_cache(pool), dev(w.q), dev(w.block_table), dev(w.ctx_lens), int(w.ctx_lens.max()), dev(w.R_k),
                        dev(w.R_v), Wo, wo_format=f, d_model=dm)
    torch.cuda.synchronize()
    ref = O.decode(pool, w.q, w.block_table, w.ctx_lens, w.R_k, w.R_v, w.W_o)
    # a folded bf16 weight is rounded once more (2^-9 of itself): of the bound's 2e-3 it uses a few parts in ten
    assert_rows_close(y.cpu().numpy(), ref, rel=4e-3 if fmt == "folded" else 2e-3, what=f"{B} {Hq} {dm} {fmt}")
