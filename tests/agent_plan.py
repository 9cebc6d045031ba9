"""The kernel and plan that the library chooses for an agent-resident call
(host only: works without a GPU)."""
import ctypes

from paper_2607_17855_amd import bi

ALGO = {"fpi": bi.BI_ALGO_FPI, "vmp": bi.BI_ALGO_VMP, "mmp": bi.BI_ALGO_MMP}


def plan_of_handle(handle, b, T, algo):
    """{"kernel": profile name, ...} of a call on a packed model, or None where
    the agent-resident family refuses it."""
    buf = ctypes.create_string_buffer(256)
    fn = bi.load().bi_test_agent_plan
    fn.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.c_char_p, ctypes.c_size_t]
    fn.restype = ctypes.c_int
    rc = fn(ctypes.c_void_p(handle), b, T, ALGO[algo], buf, 256)
    if rc == bi.BI_ERR_UNSUPPORTED:
        return None
    assert rc == bi.BI_OK, bi.bi_last_error()
    words = buf.value.decode().split()
    return {"kernel": words[0], **dict(w.split("=") for w in words[1:])}


def plan_of(model, b, T, algo):
    handle, _ = bi.bi_pack_model_host(model.n, model.U, model.K, model.deps, model.mb, model.A, model.B, model.D,
                                      bdeps=model.bdeps)
    try:
        return plan_of_handle(handle, b, T, algo)
    finally:
        bi.bi_free_model(handle)
