"""More row tiles than one grid of the fp32 attention kernel takes (2^32 threads: with 128 heads
65,536 tiles): every row is computed.  Each tile is one fragment of one token, whose row sees the
one-token prefix and itself, so the exact output is the softmax of two scores."""
import math
from types import SimpleNamespace

import numpy as np
import pytest

import paper_2511_02749_amd as spanq

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_more_tiles_than_a_grid_takes():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    frags, hq, d = 65600, 128, 64
    print(f"{frags} tiles of {hq} heads", flush=True)
    pool = spanq.Pool(num_q_heads=hq, num_kv_heads=1, head_dim=d, num_pages=frags + 8, dtype="f32", rope_theta=1e4,
                      device=0)
    tokens = np.arange(frags + 1, dtype=np.int32)
    span = lambda i: SimpleNamespace(tokens=tokens[i:i + 1], row=i)  # noqa: E731
    query = SimpleNamespace(prefix=span(0), frags=[span(1 + i) for i in range(frags)],
                            cross=SimpleNamespace(tokens=tokens[:0], row=0))
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((frags + 1, hq, d), generator=g, device="cuda")
    k, v = (torch.randn((frags + 1, 1, d), generator=g, device="cuda") for _ in range(2))
    out = torch.zeros_like(q)
    plan = pool.plan([query])
    assert plan.stats()["prefill_tiles"] == frags + 1
    plan.prefill(0, q, k, v, out)
    torch.cuda.synchronize()
    plan.destroy()
    pool.close()

    def turn(x, pos):
        a = pos * 1e4 ** (-torch.arange(d // 2, dtype=torch.float64, device="cuda") / (d // 2))
        x0, x1 = x[..., :d // 2].double(), x[..., d // 2:].double()
        return torch.cat([x0 * a.cos() - x1 * a.sin(), x1 * a.cos() + x0 * a.sin()], -1)

    qr, own = turn(q[1:], 1.0), turn(k[1:], 1.0)  # fragment tokens are at position 1, the prefix at 0
    s = torch.stack([qr @ turn(k[0, 0], 0.0), (qr * own).sum(-1)], -1) / math.sqrt(d)
    p = torch.softmax(s, -1)
    want = p[..., :1] * v[0, 0].double() + p[..., 1:] * v[1:].double()
    assert (out[1:].double() - want).abs().max() <= 1e-5
    assert torch.equal(out[0], v[0].expand(hq, d))
