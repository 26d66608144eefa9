"""The compute calls by ctypes: what binding.py takes where LORA_AMD_LIBRARY names a library and the extension module _calls has
not been built.  Same arguments and same errors; 3 to 4 us more host time a call."""
import ctypes

_P, _I, _L, _F, _Z = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t
_PROTOTYPES = [ctypes.CFUNCTYPE(ctypes.c_int, *a) for a in (
    (_P, _P), (_P, _P, _L, _P, _P, _P), (_P, _P, _P, _P, _L, _F, _P), (_P, _P, _L, _P, _P, _P, _P, _L, _F, _P),
    (_P, _P, _L, _P, _P, _P, _L, _F, _P), (_I, _I, _I, _I, _P, _L, _P, _L, _P, _L, _P),
    (_P, _P, _L, _P, _L, _P, _P, _P, _L, _P, _Z, _P), (_I, _I, _I, _I, _F, _I, _I, _P, _L, _P, _P, _P))]


def bind(check, first_stream, *addresses):
    """As that of _calls: check(status, name) raises; first_stream()[0] is torch's current stream; the functions' addresses in
    the order plan_upload, shrink, expand, delta, delta_static, base_gemm, fused_forward, merge"""
    global _check, _first_stream, _upload, _shrink, _expand, _delta, _delta_static, _base_gemm, _fused_forward, _merge
    _check, _first_stream = check, first_stream
    _upload, _shrink, _expand, _delta, _delta_static, _base_gemm, _fused_forward, _merge = (
        prototype(address) for prototype, address in zip(_PROTOTYPES, addresses))


def _ptr(obj):
    return obj if obj is None or isinstance(obj, int) else int(obj.data_ptr())


def _stream(stream):
    if stream is None:
        return _first_stream()[0]
    return stream if isinstance(stream, int) else int(stream.cuda_stream)


def lora_plan_upload(plan, stream=None):
    _check(_upload(plan.handle, _stream(stream)), "lora_plan_upload")


def lora_shrink(plan, x, ldx, d_At_ptrs, v, stream=None):
    _check(_shrink(plan.handle, _ptr(x), int(ldx), _ptr(d_At_ptrs), _ptr(v), _stream(stream)), "lora_shrink")


def lora_expand(plan, v, d_Bt_ptrs, y, ldy, beta=1.0, stream=None):
    _check(_expand(plan.handle, _ptr(v), _ptr(d_Bt_ptrs), _ptr(y), int(ldy), float(beta), _stream(stream)), "lora_expand")


def lora_delta(plan, x, ldx, d_At_ptrs, d_Bt_ptrs, v, y, ldy, beta=1.0, stream=None):
    _check(_delta(plan.handle, _ptr(x), int(ldx), _ptr(d_At_ptrs), _ptr(d_Bt_ptrs), _ptr(v), _ptr(y), int(ldy), float(beta),
                  _stream(stream)), "lora_delta")


def lora_delta_static(plan, x, ldx, d_At_ptrs, d_Bt_ptrs, y, ldy, beta=1.0, stream=None):
    _check(_delta_static(plan.handle, _ptr(x), int(ldx), _ptr(d_At_ptrs), _ptr(d_Bt_ptrs), _ptr(y), int(ldy), float(beta),
                         _stream(stream)), "lora_delta_static")


def lora_base_gemm(num_tokens, k, n, dtype, x, ldx, Wt, ldw, y, ldy, stream=None):
    _check(_base_gemm(int(num_tokens), int(k), int(n), int(dtype), _ptr(x), int(ldx), _ptr(Wt), int(ldw), _ptr(y), int(ldy),
                      _stream(stream)), "lora_base_gemm")


def lora_merge(num_layers, n, k, rank, scale, dtype, d_Wt_ptrs, ldw, d_At_ptrs, d_Bt_ptrs, variant=0, stream=None):
    _check(_merge(int(num_layers), int(n), int(k), int(rank), float(scale), int(dtype), int(variant), _ptr(d_Wt_ptrs), int(ldw),
                  _ptr(d_At_ptrs), _ptr(d_Bt_ptrs), _stream(stream)), "lora_merge")


def lora_fused_forward(plan, x, ldx, Wt, ldw, d_At_ptrs, d_Bt_ptrs, y, ldy, workspace, workspace_bytes, stream=None):
    _check(_fused_forward(plan.handle, _ptr(x), int(ldx), _ptr(Wt), int(ldw), _ptr(d_At_ptrs), _ptr(d_Bt_ptrs), _ptr(y), int(ldy),
                          _ptr(workspace), int(workspace_bytes), _stream(stream)), "lora_fused_forward")
