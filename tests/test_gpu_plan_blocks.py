"""Device blocks that a pool keeps from destroyed plans and finished decode steps for the
next ones: plans of very different sizes, made and destroyed in turn on two streams with
no synchronisation between them, give the outputs that each gives on a pool of its own."""
import dataclasses

import pytest

import paper_2511_02749_amd as spanq
import workloads as W
from tests.helpers import GpuRun

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(flush=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_blocks_pass_between_plans_of_two_streams(dtype):
    _need_gpu()
    wl = W.small_workload(dtype=dtype, prefix_len=70, frag_lens=(300, 129, 16, 90, 33, 61), frags_per_query=6,
                          n_queries=8, cross_len=40)
    queries = wl.batches[0]
    sizes = [1, 8, 2, 5, 1, 8, 3, 1, 6, 8, 2]  # queries per plan: few to many work lists and partials

    def one(run, n, out, stream=None):
        plan = run.pool.plan(queries[:n], stream)
        plan.prefill(0, run.q, run.k, run.v, out)
        plan.cross(0, run.q, run.k, run.v, out)
        plan.decode([1] * n, [q.cross.row for q in queries[:n]], stream)  # a step's block too
        plan.decode_attend(0, run.q, run.k, run.v, out)
        plan.destroy()                                 # its pages are freed, its block kept

    want = []
    for n in sizes:
        run = GpuRun(dataclasses.replace(wl, batches=[queries]))
        one(run, n, run.out)
        torch.cuda.synchronize()
        want.append(run.out.clone())
        run.close()
    # two pools' plans alternate over two streams: each pool's blocks pass between both
    runs = [GpuRun(wl), GpuRun(wl)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.zeros_like(runs[0].out) for _ in sizes]
    torch.cuda.synchronize()
    done = [None, None]  # of each pool: pages pass to its next plan, which the caller orders
    for i, n in enumerate(sizes):
        s = streams[(i // 2) % 2]
        if done[i % 2] is not None:
            s.wait_event(done[i % 2])
        one(runs[i % 2], n, outs[i], s)
        done[i % 2] = s.record_event()
    torch.cuda.synchronize()
    for i, (got, ref) in enumerate(zip(outs, want)):
        assert torch.equal(got, ref), f"plan {i} of {sizes[i]} queries"
    for run in runs:
        run.close()



@pytest.mark.parametrize("kept", [False, True])
def test_step_without_tokens_is_no_step(kept):
    """span_decode_attend after a decode step in which no query had a token: refused, whether or
    not the pool keeps a block from an earlier plan."""
    _need_gpu()
    wl = W.small_workload(n_queries=2)
    run = GpuRun(wl)
    if kept:
        run.run_batch(wl.batches[0]).destroy()
    plan = run.pool.plan(wl.batches[0])
    if kept:
        run.pool.plan(wl.batches[0][:1]).destroy()
    torch.cuda.synchronize()
    plan.decode([0] * len(wl.batches[0]), [0] * len(wl.batches[0]))
    with pytest.raises(spanq.SpanError) as ei:
        plan.decode_attend(0, run.q, run.k, run.v, run.out)
    assert ei.value.code == -4
    plan.destroy()
    run.close()
