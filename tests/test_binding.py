"""The native half of the Python binding refuses arguments that do not fit before anything is enqueued.  No GPU needed."""
import pytest
import torch


@pytest.mark.parametrize("call,error", [
    (lambda s, x, bm, v, ro: s.linear(x, bm, v, ro, None, None), TypeError),                                     # host tensors
    (lambda s, x, bm, v, ro: s.linear(x[0], bm, v, ro, None, None), ValueError),                                 # x is no matrix
    (lambda s, x, bm, v, ro: s.linear(3, bm, v, ro, None, None), TypeError),                                     # no tensor
    (lambda s, x, bm, v, ro: s.salr_sparse_lowrank_linear(x, bm, v, ro, None, None, x[:1, :2].clone(), None), ValueError),
    (lambda s, x, bm, v, ro: s.salr_sparse_lowrank_linear(x, bm, v, ro[:2], None, None, x[:, :3].clone(), None), ValueError),
    (lambda s, x, bm, v, ro: s.salr_sparse_lowrank_linear(x, bm, v, ro, x[:2, :4].clone(), x[:, :3].clone(), x[:, :3].clone(),
                                                          None), ValueError),                                    # adapter shapes
    (lambda s, x, bm, v, ro: s.linear_prepared(x, bm, v, ro, None, None, None), (TypeError, ValueError)),
    (lambda s, x, bm, v, ro: s.salr_qsalr_linear(x, bm, v, v, ro[:1], 8, None, None, x[:, :3].clone(), None), ValueError),
    (lambda s, x, bm, v, ro: s.linear_backward(x[:, :8].clone(), x[:, :3].clone(), bm, v, ro, None, None), (TypeError, ValueError)),
])
def test_bad_arguments(call, error):
    import paper_2601_16991_amd as salr
    x = torch.zeros(2, 64, dtype=torch.int16)
    bm, v, ro = torch.zeros(3, 2, dtype=torch.int32), torch.zeros(8, dtype=torch.int16), torch.zeros(4, dtype=torch.int32)
    with pytest.raises(error):
        call(salr, x, bm, v, ro)
