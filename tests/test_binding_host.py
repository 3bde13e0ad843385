"""The binding's checks of its tensor arguments, on a host without a GPU."""
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("symbol", [True, False], ids=["with raw streams", "without"])
def test_host_tensors_are_refused_by_any_torch(monkeypatch, symbol):
    """Host tensors raise ValueError, also under a torch built without GPU
    support, which lacks the symbol that reads a raw stream."""
    import paper_2205_14473_amd as E
    from paper_2205_14473_amd import _binding
    for name in ("_torch", "_F32", "_U64", "_raw_stream", "_device"):
        monkeypatch.setattr(_binding, name, None)
    if not symbol:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    t = torch.zeros(8)
    with pytest.raises(ValueError, match="device tensors"):
        E.ea_toy_grad(4, 2, t, t, t, t, t, t, t)
    with pytest.raises(ValueError, match="device tensors"):
        E.ea_step(E.Config(d=8, N=1), 1, *[t] * 13)
