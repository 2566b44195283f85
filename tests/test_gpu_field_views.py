"""The views of a batch's state: of the state itself, each caller's own, also where a field is first asked for in inference mode;
calls go to the current stream."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


def test_fields_are_views_of_the_state_on_any_stream():
    s = synth.CONFIGS["tiny_f32"]
    m = S.Model.from_shape(s, max_pos=64)
    m.set_embed(torch.randn(s.vocab, s.d_model, device="cuda"))
    b = S.Batch(m, 5)
    with torch.inference_mode():
        b.field("h")
    for name in S._FIELD_TYPES:
        v, off = b.field(name), getattr(b.layout, name)
        assert v.data_ptr() == b.state.data_ptr() + off and v.dtype == S._FIELD_TYPES[name]
        shape, changed = v.shape, b.field(name)
        changed.unsqueeze_(0)                                # in place, of this view alone
        assert v.shape == shape and b.field(name).shape == shape and b.field(name).is_contiguous()
        if v.is_floating_point():
            b.field(name).requires_grad_()
            assert not b.field(name).requires_grad
    assert b.field("h").shape == (5, s.d_model) and b.field("tok_in").shape == (5,) and b.field("status").shape == (1,)
    b.reset(np.arange(5), np.zeros(5, np.int32))
    side = torch.cuda.Stream()
    assert S._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert S._stream() == side.cuda_stream
        b.begin_step()
    side.synchronize()
    b.field("h").mul_(2.0)                                   # in place, outside inference mode, and seen by the state
    h = b.state[b.layout.h:b.layout.h + 5 * s.d_model * 4].view(torch.float32).view(5, -1)
    assert torch.equal(h, 2.0 * m._keep["embed"][:5])
