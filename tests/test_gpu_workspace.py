"""The workspace that the binding keeps by itself: one for each stream, replaced by a larger one where a call needs it.  (A call
with a stream argument is not given a guarded workspace by the fixture of conftest.py.)"""
import pytest
import torch

from test_gpu_parity import _pk

pytestmark = pytest.mark.gpu

L, H, D, T, GROUP = 1, 4, 128, 1100, 4


def _pool():
    g = torch.Generator(device="cuda").manual_seed(9)
    pool = _pk().Pool(L, H, D, T).bind()
    K, V = (torch.randn((L, H, T, D), device="cuda", generator=g).half() for _ in range(2))
    pool.encode(K, V)
    Q = torch.randn((L, 20, 1, H * GROUP, D), device="cuda", generator=g).half()
    torch.cuda.synchronize()
    return pool, Q[:, :2].contiguous(), Q


def _streams():
    return {"current": torch.cuda.current_stream(), "side": torch.cuda.Stream()}


@pytest.mark.parametrize("which", ["current", "side"])
def test_a_small_call_a_larger_one_and_the_small_one_again(which):
    pool, small, large = _pool()
    stream = _streams()[which]
    want_small, want_large = pool.attend(small, splits=2), pool.attend(large, splits=4)
    torch.cuda.synchronize()
    sizes = []
    for Q, splits, want in ((small, 2, want_small), (large, 4, want_large), (small, 2, want_small)):
        out = torch.empty(Q.shape, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        pool.attend(Q, out, splits=splits, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        sizes.append(pool._workspaces[stream.cuda_stream].numel())
    assert sizes[0] == pool.attend_workspace_bytes(small, splits=2)
    assert sizes[1] == sizes[2] == pool.attend_workspace_bytes(large, splits=4) > sizes[0]
    assert list(pool._workspaces) == [stream.cuda_stream]


@pytest.mark.parametrize("which", ["current", "side"])
def test_calls_that_are_refused(which):
    pk = _pk()
    pool, small, large = _pool()
    stream = _streams()[which]
    odd = small[..., :6, :].contiguous()                 # six query heads over four KV heads
    with pytest.raises(pk.PolyKVError) as e:             # no workspace yet
        pool.attend(odd, stream=stream)
    assert e.value.status == pk.ESHAPE and not pool._workspaces
    pool.attend(small, stream=stream)
    kept = pool._workspaces[stream.cuda_stream]
    with pytest.raises(pk.PolyKVError) as e:
        pool.attend(odd, stream=stream)
    assert e.value.status == pk.ESHAPE
    given = torch.empty(pool.attend_workspace_bytes(large, splits=4) - 1, dtype=torch.uint8, device="cuda")
    with pytest.raises(pk.PolyKVError) as e:             # too small, and not the binding's to replace
        pool.attend(large, splits=4, stream=stream, workspace=given)
    assert e.value.status == pk.ENOMEM and pool._workspaces[stream.cuda_stream] is kept
    torch.cuda.synchronize()


def test_a_replaced_workspace_stays_with_its_stream():
    """Work of that stream may still use it: its memory must not go to the next tensor of another stream."""
    pool, small, large = _pool()
    side = torch.cuda.Stream()
    pool.attend(small, splits=2, stream=side)
    torch.cuda.synchronize()
    old = pool._workspaces[side.cuda_stream]
    at, n = old.data_ptr(), old.numel()
    del old
    pool.attend(large, splits=4, stream=side)
    others = [torch.empty(n, dtype=torch.uint8, device="cuda") for _ in range(64)]
    assert pool._workspaces[side.cuda_stream].data_ptr() != at and all(t.data_ptr() != at for t in others)
    torch.cuda.synchronize()
