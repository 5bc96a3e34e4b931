"""Attention kernels that take any number of query heads per kv head (fp32 pools, and
bf16 pools outside the tiled kernels' head counts) against the oracle, at the edges of
their tiles: 1 to 130 heads per kv head (130 is two chunks of 128), row tiles of one
token, one 16- or 32-row block and one row more, key lists of one page, of a partial
page and of many splits; cold, then every fragment cached in another order (each read
at a position other than its own), then decode steps.

Tolerances as everywhere (max abs error): 1e-4 for fp32 pools, 2e-2 for bf16 pools."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import TOL, GpuRun, check_rows, computed_rows
from tests.test_decode import _cut, _decode_through

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HEADS = [(3, 1, 128), (6, 2, 64), (5, 1, 64), (14, 2, 128), (24, 1, 128), (130, 1, 64)]
CASES = ([("bf16", *h) for h in HEADS] + [("f32", 3, 1, 128), ("f32", 7, 1, 64), ("f32", 2, 2, 128)])


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(flush=True)


@pytest.mark.parametrize("cross", [1, 17, 70])
@pytest.mark.parametrize("dtype,hq,hkv,d", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_cold_cached_and_decoded_rows(dtype, hq, hkv, d, cross):
    wl = W.small_workload(dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=33,
                          frag_lens=(37, 64, 1, 130, 16), frags_per_query=5, n_queries=2, cross_len=cross + 20,
                          orders=[[0, 1, 2, 3, 4], [4, 3, 1, 0, 2]], batch_split=[1, 1])
    run = GpuRun(wl, nan_pool=True)
    first = run.run_batch([_cut(q, cross) for q in wl.batches[0]])
    check_rows(run, wl.batches[0], computed_rows(first), TOL[dtype], limit=400)
    full = wl.batches[1]
    plan = run.run_batch([_cut(q, cross) for q in full], commit=False)
    assert plan.stats()["tokens_new"] == 0
    check_rows(run, full, plan.rows()[1], TOL[dtype])
    _decode_through(run, plan, full, cross, [[1], [19]])
    plan.destroy()
    run.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_at_addresses_aligned_to_an_element_only(dtype):
    """q and out one element past an aligned address: the rows are read and written there."""
    wl = W.small_workload(dtype=dtype, n_q_heads=6, n_kv_heads=2, head_dim=64, cross_len=20)
    run = GpuRun(wl)
    plan = run.run_batch(wl.batches[0], commit=False)
    want = run.out.clone()

    def shifted(t):
        flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        flat[1:] = t.flatten()
        return flat[1:].view(t.shape)

    q, out = shifted(run.q), shifted(torch.zeros_like(run.out))
    plan.prefill(0, q, run.k, run.v, out)
    plan.cross(0, q, run.k, run.v, out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    plan.destroy()
    run.close()
