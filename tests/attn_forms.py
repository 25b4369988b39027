"""The forms the attention kernel comes in (query rows per workgroup, groups of its wavefronts that split the keys, from
queues or one workgroup per block), and a call in a form named by the test through the library's internal entry: the
public calls choose the form by size, and at the sizes of most tests would always choose the same one."""
import ctypes as C

import torch

import paper_2505_21036_amd as rf

_ROWS = [(64, 4, 0), (64, 2, 0), (128, 1, 0), (256, 1, 0), (256, 1, 1), (384, 1, 1)]


def forms(D, room=True):
    """Forms of head_dim D; room: with those that walk copies of K and V."""
    there = [f for f in _ROWS if not (D == 64 and f == (256, 1, 0))]
    return there if room else [f for f in there if not needs_copies(D, f)]


def needs_copies(D, form):
    return form == ((256, 1, 1) if D == 64 else (384, 1, 1))


def attention_as(form, Q, K, V, head_class, layout, params=None, out=None, workspace=None, head_bw=None, bandwidths=None):
    """rf_sparse_attention(_plus) in `form`; workspace as there."""
    B, nH, _, D = Q.shape
    out = torch.empty_like(Q) if out is None else out
    if workspace is None:
        workspace = torch.empty(rf.RF_ATTENTION_MIN_WORKSPACE, dtype=torch.uint8, device=Q.device)
    f = rf.load_library().rf_internal_attention_as
    f.restype, vp = C.c_int, C.c_void_p
    f.argtypes = [C.c_int] * 3 + [vp] * 5 + [vp] + [C.c_int] * 4 + [vp] * 4 + [C.c_size_t, vp]
    bws = None if bandwidths is None else (C.c_float * len(bandwidths))(*bandwidths)
    st = f(*form, Q.data_ptr(), K.data_ptr(), V.data_ptr(), None if head_class is None else head_class.data_ptr(),
           None if head_bw is None else head_bw.data_ptr(), bws, 0 if bws is None else len(bandwidths), B, nH, D,
           C.cast(C.byref(layout), vp), None if params is None else C.cast(C.byref(params), vp), out.data_ptr(),
           workspace.data_ptr(), workspace.numel(), torch.cuda.current_stream().cuda_stream)
    if st != 0:
        raise rf.RfError(st, "rf_internal_attention_as")
    return out
