"""Merging of KV splits: part counts below, at and above the four parts a thread has in
flight and its multiples (with and without several threads per row), on row tiles of 256
rows whose last splits lie past their first rows (a row that sees no key of a part skips
it), for fp16 and fp32 partials, against the oracle.

Tolerances as everywhere (max abs error): 1e-4 for fp32 pools, 2e-2 for bf16 pools."""
import pytest

import workloads as W
from tests.helpers import TOL, GpuRun, check_rows

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(flush=True)


@pytest.mark.parametrize("frags", [1, 2, 3, 4, 5, 8, 9, 18])
@pytest.mark.parametrize("dtype,hq,hkv,d,cross", [("bf16", 1, 1, 64, 250), ("bf16", 4, 1, 128, 70), ("bf16", 4, 1, 64, 3),
                                                  ("f32", 2, 1, 128, 40), ("f32", 1, 1, 64, 1)])
def test_part_counts(dtype, hq, hkv, d, cross, frags):
    wl = W.small_workload(dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=64,
                          frag_lens=(256,) * frags, frags_per_query=frags, n_queries=1, cross_len=cross,
                          orders=[list(range(frags))], batch_split=[1])
    run = GpuRun(wl, nan_pool=True)
    plan = run.run_batch(wl.batches[0])
    check_rows(run, wl.batches[0], plan.rows()[1], TOL[dtype])
    plan.destroy()
    run.close()
