"""Infinite and NaN values in the kernels for any number of query heads per kv head (fp32
pools, and bf16 pools outside the tiled kernels): a value reaches the rows that see some key
of its page, and no other row: every row before the page has the bits it has with a finite
value there.  Prefill rows, cross rows (row tiles that do not start at a page) and the rows of
one decode step that starts inside a page."""
import numpy as np
import pytest

import workloads as W
from tests.helpers import GpuRun
from tests.test_decode import _cut

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [("bf16", 3, 1, 128), ("bf16", 6, 2, 64), ("bf16", 24, 1, 128), ("bf16", 130, 1, 64), ("f32", 3, 1, 128),
         ("f32", 2, 2, 64)]


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype,hq,hkv,d", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_rows_before_a_page_do_not_meet_its_values(dtype, hq, hkv, d, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c0, cross = 10, 60
    wl = W.small_workload(dtype=dtype, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefix_len=33, frag_lens=(100,),
                          frags_per_query=1, n_queries=1, cross_len=cross)
    query = wl.batches[0][0]
    frag, own = query.frags[0].row, query.cross.row

    def outputs(at=None, decode=False):
        """Output rows of the query with `value` as the value of caller row `at`."""
        run = GpuRun(wl)
        if at is not None:
            bits = {"bf16": (torch.bfloat16, torch.int16), "f32": (torch.float32, torch.float32)}[dtype]
            run.v[at] = torch.tensor(value, dtype=bits[0], device="cuda").view(bits[1])
        plan = run.run_batch([_cut(query, c0 if decode else cross)], commit=False)
        if decode:
            plan.decode([cross - c0], [own + c0])
            plan.decode_attend(0, run.q, run.k, run.v, run.out)
            torch.cuda.synchronize()
        out = run.out_rows(np.arange(run.out.shape[0]))
        plan.destroy()
        run.close()
        return out

    clean, decoded = outputs(), outputs(decode=True)
    for first, n, want, decode in ((frag, 100, clean, False), (own, cross, clean, False), (own, cross, decoded, True)):
        for t in (17, 40, 59):
            print(dtype, hq, hkv, d, value, "row", t, "of", n, "decode" if decode else "", flush=True)
            got = outputs(first + t, decode)
            page = t // 16 * 16
            assert np.array_equal(got[first:first + page], want[first:first + page])
            assert not np.isfinite(got[first + t]).any()
            assert np.array_equal(got[:frag], want[:frag])  # the prefix
