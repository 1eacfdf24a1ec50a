"""The Python entry points on device tensors that share storage."""
import pytest
import torch

from _util import dev

pytestmark = pytest.mark.gpu


def test_results_in_a_lazy_clone_leave_its_original_alone():
    """An output that is a copy-on-write clone gets storage of its own before it is written, as with Tensor.data_ptr()."""
    import paper_2310_06993_amd.binding as b
    x = torch.randn(4096, device=dev())
    original = torch.zeros(4096, device=dev())
    out = torch._lazy_clone(original)
    want = torch.empty(4096, device=dev())
    b.or_rht_encode(x, 4096, 10, 1, want)
    b.or_rht_encode(x, 4096, 10, 1, out)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and not bool(original.any())
    # and an input that is one is read as it is
    again = torch.empty(4096, device=dev())
    b.or_rht_encode(torch._lazy_clone(x), 4096, 10, 1, again)
    assert torch.equal(again, want)
