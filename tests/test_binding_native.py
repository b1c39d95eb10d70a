"""The binding's native half takes over a call only where binding.py's own
checks accept it: it returns None for anything it cannot vouch for."""
import pytest
import torch

DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    from paper_2310_08152_amd import binding
    return binding


def test_native_half_defers_without_a_gpu_tensor(B):
    nat = B._nat()
    x = torch.zeros(4, dtype=torch.int32)
    assert nat.kv_commit(x, x, x, x, x, x, 1, 1, 1, None, None) is None      # host tensors
    assert nat.kv_commit(x, x) is None                                       # too few
    assert nat.kv_commit(None, x, x, x, x, x, 1, 1, 1, None, None) is None   # missing
    assert nat.sckv_prefill_plan(x, "4", 1, 1, x, None) is None              # not a number
    assert nat.sckv_prefill_plan(x, 1 << 40, 1, 1, x, None) is None          # above int32
    with pytest.raises(B.SckvError):
        B.kv_commit(x, x, x, x, x, x, 1, 1, 1)


FORMS = {
    # name: (x, b, H, n, stride) for rope_apply with d = 64
    "four-dim": lambda z: (z(2, 3, 8, 64), 2, 3, 8, 512),
    "row-slice": lambda z: (z(2, 3, 8, 64)[:, :, 2:6], 2, 3, 4, 512),
    "contiguous-3d": lambda z: (z(6, 8, 64), 2, 3, 8, 512),
    "one-batch-any-stride": lambda z: (z(2, 3, 8, 64)[1:], 1, 3, 8, 512),
    "one-row-any-row-stride": lambda z: (z(2, 3, 8, 128)[:, :, ::8, :64], 2, 3, 1, 1024),
    "wrong-stride": lambda z: (z(2, 3, 8, 64), 2, 3, 8, 576),
    "transposed-heads": lambda z: (z(2, 8, 3, 64).transpose(1, 2), 2, 3, 8, 512),
    "past-the-storage": lambda z: (z(2, 3, 4, 64), 2, 3, 8, 512),
    "offset-past-the-storage": lambda z: (z(7, 512)[1:, 64:], 2, 3, 8, 512),
    "float64": lambda z: (z(2, 3, 8, 64).double(), 2, 3, 8, 512),
    "unsupported-head": lambda z: (z(2, 3, 8, 64), 2, 3, 8, 500),
}


@pytest.mark.gpu
@pytest.mark.parametrize("form", list(FORMS))
def test_native_and_python_checks_agree(B, form, monkeypatch):
    """Both halves accept or refuse a form alike, with the same outputs."""
    print(f"binding form={form}", flush=True)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

    def z(*shape):
        g = torch.Generator(device=DEV).manual_seed(3)
        return torch.randn(shape, generator=g, device=DEV).to(torch.bfloat16)

    class Deferring:
        def __getattr__(self, name):
            return lambda *a: None

    got = []
    for native in (True, False):
        if not native:
            monkeypatch.setattr(B, "_native", Deferring())
        x, b, H, n, stride = FORMS[form](z)
        y = torch.zeros(b * H * stride, dtype=x.dtype, device=DEV)
        try:
            B.rope_apply(x, y, b, H, n, stride, stride, 64, None, 16, 0, 0.0)
            torch.cuda.synchronize()
            got.append(("ok", y.cpu()))
        except B.SckvError as e:
            got.append((e.code, None))
    assert got[0][0] == got[1][0], got
    if got[0][1] is not None:
        assert torch.equal(got[0][1], got[1][1])


@pytest.mark.gpu
def test_native_half_keeps_positions_required(B):
    """A rotary base that is not zero needs positions, also one that rounds to
    zero in 32 bits."""
    print("binding theta", flush=True)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.zeros(1, 1, 4, 64, device=DEV)
    for theta in (1e-60, 1e4):
        assert B._nat().rope_apply(x, x, 1, 1, 4, 256, 256, 64, None, 4, 0, theta, None) is None
        with pytest.raises(B.SckvError) as e:
            B.rope_apply(x, x, 1, 1, 4, 256, 256, 64, None, 4, 0, theta)
        assert e.value.code == B.EINVAL
