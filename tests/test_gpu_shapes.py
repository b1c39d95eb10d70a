"""GPU launch shapes against the CPU oracle, at the sizes where a launch
changes: counts of (sequence, head) slices around the multiples of 8 that the
work order deals to the XCDs."""
import numpy as np
import pytest
import torch

from oracle import sckv_oracle as O

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# the output's bf16 rounding (2^-9 of values below 4) and that of the
# probabilities (2^-9 of each, values below 5) stay under half of this
TOL = 2e-2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_08152_amd import binding  # noqa: F401  (fails loudly without the library)


def P():
    from paper_2310_08152_amd import path
    return path


def W():
    from paper_2310_08152_amd import workload
    return workload


def f64(t):
    return t.detach().to("cpu", torch.float64).numpy()


def rnd(shape, seed, dtype="bf16"):
    return W().randn(shape, seed=seed, dtype=dtype).to(DEV)


@pytest.mark.parametrize("b,H", [(1, 1), (1, 7), (2, 4), (3, 3), (1, 17), (5, 16)])
def test_prefill_covers_every_slice(b, H):
    """Every slice's every block is computed whatever the number of slices
    (left-over slices alone, whole groups alone, both, a partial group)."""
    print(f"prefill b={b} H={H}", flush=True)
    L, d = 300, 64
    rng = np.random.default_rng(b * 100 + H)
    spans = [W().spans_uniform_lengths(L, 0.4, 4, 24, rng) for _ in range(b)]
    q, k, v = (rnd((b, H, L, d), 200 + i) for i in range(3))
    o = torch.full_like(q, float("nan"))
    P().prefill_layer(q, k, v, o, P().SpanMeta(spans, L, DEV), P().Workspace(b, H, L, L, d, DEV), L)
    torch.cuda.synchronize()
    Q, K, V, Og = f64(q), f64(k), f64(v), f64(o)
    assert np.isfinite(Og).all()
    for s in range(b):
        ref = O.masked_attention(Q[s], K[s], V[s], O.attention_mask(O.token_types(spans[s], L)))
        assert np.abs(Og[s] - ref).max() <= TOL, s
