"""The sampled space with other tables than the workload's: tensor-parallel degrees that are no powers of two (their
division is not a product with a reciprocal), odd block sizes, budgets and KV-head choices, both time models."""
import dataclasses

import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge

pytestmark = pytest.mark.gpu
u32 = lambda *v: np.array(v, dtype=np.uint32)                              # noqa: E731


@pytest.mark.parametrize("tp,blk,mbt,kvc", [((3, 5, 6, 7), (7, 24), (400, 1000, 8001), (1, 3, 5, 0)),
                                            ((1, 2, 4, 16), (1, 4096), (300, 40000, 2048), (8, 8, 1000, 2)),
                                            ((1, 1, 1, 12), (16, 32), (2048, 4096, 8192), (0, 0, 0, 0))])
@pytest.mark.parametrize("tm", [0, 1])
def test_tables(ora, tp, blk, mbt, kvc, tm):
    import torch
    sp = dataclasses.replace(wl.sample_space(), tp=u32(*tp), kv_block=u32(*blk), mbt=u32(*mbt), kv_choices=u32(*kvc))
    ctx = guide.Context(0)
    n, first, seed = 4_011, (1 << 40) + 5, 0xFEDCBA9876543210
    out = bridge.metric_buffers(n, names=("t_prefill", "t_batch", "cost", "b_max", "feasible", "bucket"))
    out.update(feasible_count=torch.zeros(1, dtype=torch.int64, device="cuda"),
               win_val=torch.zeros(10, dtype=torch.float64, device="cuda"),
               win_idx=torch.zeros(10, dtype=torch.int64, device="cuda"), hist=torch.zeros(256, dtype=torch.int64, device="cuda"))
    ctx.eval_sampled(bridge.gpu_space(sp), seed, first, n, wl.BUCKET_EDGES, 1.0, out, time_model=tm)
    torch.cuda.synchronize()
    exp = ora.eval_sampled(bridge.ora_space(sp), seed, first, n, wl.BUCKET_EDGES, 1.0, time_model=tm, columns=True)
    for k in ("t_prefill", "t_batch", "cost"):
        assert bridge.rel_err(out[k].cpu().numpy(), exp[k]).max() <= 1e-9, k
    np.testing.assert_array_equal(bridge.to_np(out["b_max"], np.uint32), exp["b_max"])
    np.testing.assert_array_equal(out["feasible"].cpu().numpy(), exp["feasible"])
    np.testing.assert_array_equal(bridge.to_np(out["bucket"], np.uint32), exp["bucket"])
    assert int(out["feasible_count"].item()) == int(exp["feasible_count"])


# Around a block and past every resident block; feed-forward ratios in floating point, in integers, wrapped to 32 bits; edges in no
# order, some twice, none at all, and such that are no numbers or infinite.
EDGES = (8.0e9, 1.0e9, 3.0e9, 3.0e9, 1.0e30, 2.0e10, 5.0e11, 7.0e9, 1.0, 1.0e12, 4.0e9, 2.0e9, 6.0e9, 9.0e9, 1.0e10)      # a bucket is a count
ODD_EDGES = (np.inf, 3.0e9, np.nan, -np.inf, 2.0e10, -np.nan, 7.0e9)


@pytest.mark.parametrize("n,columns,ffn,edges", [(1, True, (5, 3), EDGES), (511, False, (5, 3), EDGES), (513, True, (32767, 32768), EDGES),
                                                 (1023, True, (70000, 1), EDGES), (1023, True, (32767, 32767), EDGES),
                                                 (512 * 512 + 1, False, (5, 3), EDGES), (2000, True, (5, 3), ODD_EDGES),
                                                 (2000, False, (5, 3), (np.nan,) * 15), (2000, True, (5, 3), ())])
@pytest.mark.parametrize("tm", [0, 1])
def test_block_edges_and_ratios(ora, n, columns, ffn, edges, tm):
    import torch
    sp = dataclasses.replace(wl.sample_space(), ffn_lo_x2=ffn[0], ffn_span_x2=ffn[1])
    ctx = guide.Context(0)
    out = bridge.metric_buffers(n, names=("t_prefill", "t_batch", "cost", "b_max", "feasible", "bucket")) if columns else {}
    nb = len(edges) + 1
    out.update(feasible_count=torch.full((1,), -1, dtype=torch.int64, device="cuda"),
               win_val=torch.full((nb,), -1.0, dtype=torch.float64, device="cuda"),
               win_idx=torch.full((nb,), -1, dtype=torch.int64, device="cuda"),
               hist=torch.full((256,), -1, dtype=torch.int64, device="cuda"))
    ctx.eval_sampled(bridge.gpu_space(sp), 77, 12345, n, edges, 5.0, out, time_model=tm)
    torch.cuda.synchronize()
    exp = ora.eval_sampled(bridge.ora_space(sp), 77, 12345, n, edges, 5.0, time_model=tm, columns=True)
    assert int(out["feasible_count"].item()) == int(exp["feasible_count"]) == int(out["hist"].sum().item())
    np.testing.assert_array_equal(bridge.to_np(out["win_idx"], np.uint64), exp["win_idx"])
    win_val, empty = out["win_val"].cpu().numpy(), exp["win_idx"] == np.iinfo(np.uint64).max
    assert (win_val[empty] == np.inf).all() and (bridge.rel_err(win_val[~empty], exp["win_val"][~empty]) <= 1e-9).all()
    np.testing.assert_array_equal(bridge.to_np(out["hist"], np.uint64), exp["hist"])
    if columns:
        for k in ("t_prefill", "t_batch", "cost"):
            assert bridge.rel_err(out[k].cpu().numpy(), exp[k]).max() <= 1e-9, k
        np.testing.assert_array_equal(bridge.to_np(out["bucket"], np.uint32), exp["bucket"])
        np.testing.assert_array_equal(bridge.to_np(out["b_max"], np.uint32), exp["b_max"])
        np.testing.assert_array_equal(out["feasible"].cpu().numpy(), exp["feasible"])
