"""Device of the segment table: its three offsets lie together on the device
asked for, wherever the caller's offsets were."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["cpu", "cuda", "cuda:0", None])
@pytest.mark.parametrize("given", ["cpu", "cuda"])
@pytest.mark.parametrize("two", [False, True])
def test_offsets_on_the_device_asked_for(where, given, two):
    import paper_2011_11134_amd as dg
    want = torch.device("cpu" if where == "cpu" else "cuda:0")
    a = torch.tensor([0, 3, 3, 10], device=given)
    b = torch.tensor([0, 2, 7, 11], device=given) if two else None
    d_a, d_b, d_o, nseg, total, _, _ = dg.segments(10, 11 if two else 10, a, b,
                                                   self_pairs=not two, device=where)
    assert [t.device for t in (d_a, d_b, d_o)] == [want] * 3
    nb = [2, 5, 4] if two else [3, 0, 7]
    size = [n * m for n, m in zip([3, 0, 7], nb)]
    assert d_a.tolist() == a.tolist() and d_b.tolist() == (b if two else a).tolist()
    assert d_o.tolist() == [0, size[0], size[0] + size[1]] and (nseg, total) == (3, sum(size))
