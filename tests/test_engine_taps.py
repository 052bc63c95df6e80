"""The engine's views of the workspace, without a GPU."""
import pytest
import torch

from paper_2602_01274_amd import binding as B
from paper_2602_01274_amd.engine import Session


def test_tap_views_are_the_callers_own(monkeypatch):
    """Two looks at a buffer share its memory and nothing else: a change of shape or flags in place stays with the tensor it
    was made on."""
    s = Session.__new__(Session)
    s.max_batch, s.G1, s.V, s.ctx, s._taps = 3, 2, 4, None, {}
    s.ws_view = torch.arange(3 * 2 * 4, dtype=torch.float32).view(torch.uint8)
    nb = 2 * 4 * 4

    def peek(ctx, seq, what):
        if not 0 <= seq < 3:
            raise B.PacerError(B.EINVAL, "peek: bad arguments")
        return s.ws_view.data_ptr() + seq * nb, nb
    monkeypatch.setattr(B, "pacer_peek", peek)
    a, b = s.draft_logits(1), s.draft_logits(1)
    assert a is not b and a.data_ptr() == b.data_ptr() and a.tolist() == [[8, 9, 10, 11], [12, 13, 14, 15]]
    a.unsqueeze_(0)
    b.requires_grad_()
    c = s.draft_logits(1)
    assert c.shape == (2, 4) and not c.requires_grad
    c[0, 0] = -1.0
    assert s.draft_logits(1)[0, 0] == -1.0
    for bad in (-1, 3):
        with pytest.raises(B.PacerError):
            s.draft_logits(bad)
    s.__dict__.clear()
    s.ctx = None
