"""One GEMM on a kernel the test names (the library's internal entry for tests)."""
import ctypes

from paper_2608_01785_amd import binding

RESID, SWIGLU, QKV, GATED, GELU = 1, 2, 3, 4, 5
SKINNY, PERSISTENT = -2, -1
TILES = range(7)

FIELDS = ("A", "W", "w_f16", "M", "K", "N", "out", "out_f32", "ldo", "resid", "resid_f32", "ffn", "q", "k", "v", "pos",
          "pos_stride", "sec1", "sec2", "k_off", "v_off", "kv_head_stride", "rope", "bias", "gate", "gate_stride",
          "row_seq", "hq", "hkv", "dh", "part", "counters", "k8_rows", "clock", "w_resident")


def choice(M, N, K, cus):
    """The kernel the dispatch takes for a prefill-sized product."""
    return binding.lib().hs_gemm_choice(M, N, K, cus)


def call(epi, kernel, cus=256, stream=None, **args):
    """A launch, ready to be made: tensors and numbers by field name, missing ones zero.  stream: a handle, or the
    default stream."""
    unknown = set(args) - set(FIELDS)
    assert not unknown, unknown
    vals = [args.get(f, 0) for f in FIELDS]
    for t in vals:
        assert isinstance(t, int) or (t.is_cuda and t.is_contiguous())
    arr = (ctypes.c_int64 * len(FIELDS))(*[t if isinstance(t, int) else t.data_ptr() for t in vals])
    fn = binding.lib().hs_gemm_direct
    fn.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p]

    def launch():
        binding._check(fn(epi, kernel, cus, arr, len(FIELDS), stream))
    launch.tensors = vals   # alive as long as the call
    return launch


def run(epi, kernel, cus=256, **args):
    call(epi, kernel, cus, **args)()


def panels(w):
    """[N, K] -> [K / 32][N][32], the order of prepared fp16 weights."""
    n, k = w.shape
    return w.reshape(n, k // 32, 32).transpose(0, 1).contiguous()
