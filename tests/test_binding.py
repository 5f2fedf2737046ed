"""The binding's argument handling: kept descriptors equal fresh ones for every size, type and
option that enters them, and tensors that the calls refuse are still refused."""
import math

import pytest
import torch

import paper_2606_01774_amd as bd


def _fields(desc):
    return {name: getattr(desc, name) for name, _ in desc._fields_}


@pytest.mark.parametrize("dtype,out_dtype", [(torch.bfloat16, torch.float32), (torch.bfloat16, torch.bfloat16),
                                             (torch.float32, torch.float32), (torch.float16, torch.float64)])
@pytest.mark.parametrize("shape,h_v,d_v,block,scale,num_seqs,route", [
    ((2, 96, 1, 64), 3, 128, 16, None, 0, bd.BDGDN_ROUTE_FUSED),
    ((1, 96, 2, 128), 2, 64, 32, 0.25, 3, bd.BDGDN_ROUTE_RECORDS),
])
def test_kept_descriptors_equal_fresh_ones(dtype, out_dtype, shape, h_v, d_v, block, scale, num_seqs, route):
    q, v = torch.empty(shape, dtype=dtype), torch.empty(*shape[:2], h_v, d_v, dtype=dtype)
    fresh = bd.make_fwd_desc(q, v, block=block, scale=scale, num_seqs=num_seqs, route=route, out_dtype=out_dtype)
    plan = bd._fwd_desc(q, v, block, scale, num_seqs, out_dtype, route)
    assert _fields(plan[0]) == _fields(fresh)
    for query in (bd.bdgdn_fwd_train_workspace, bd.bdgdn_bwd_train_workspace):
        assert bd._plan_bytes(plan, query) == bd._plan_bytes(plan, query) == query(fresh)
    R, L, h_qk, d_k = shape
    serve = bd._serve_desc(q, v, scale, out_dtype)._obj
    assert _fields(serve) == _fields(bd.ServeDesc(R, h_qk, h_v, d_k, d_v, L,
                                                  1 / math.sqrt(d_k) if scale is None else scale,
                                                  bd._DT.get(dtype, -1), bd._DT.get(out_dtype, -1)))
    x, w = torch.empty(shape[:3], dtype=dtype), torch.empty(shape[2], 4)
    conv = bd._conv_desc(x, w, block, bd.BDGDN_ACT_NONE, num_seqs)[0]
    assert _fields(conv) == _fields(bd.make_conv_desc(x, w, block=block, activation=bd.BDGDN_ACT_NONE,
                                                      num_seqs=num_seqs))


@pytest.mark.parametrize("value,dtype", [(torch.zeros(4), None), ([1.0], None), (torch.zeros(4, 4).t(), torch.float32)])
def test_unusable_tensors_are_refused(value, dtype):
    with pytest.raises(ValueError, match="x must be a device tensor"):
        bd._p(value, "x", dtype)
    assert bd._p(None, "x", dtype) is None


@pytest.mark.gpu
def test_device_tensors_of_another_type_or_stride_are_refused():
    x = torch.zeros(4, 2, device="cuda")
    assert bd._p(x, "x", torch.float32) == x.data_ptr() == bd._p(torch.nn.Parameter(x), "x", torch.float32)
    with pytest.raises(ValueError, match="must be torch.int32"):
        bd._p(x, "x", torch.int32)
    with pytest.raises(ValueError, match="must be contiguous"):
        bd._p(x.t(), "x", torch.float32)
