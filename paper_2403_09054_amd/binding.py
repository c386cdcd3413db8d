"""ctypes binding of libkeyformer.so: same names as the C ABI, marshalling only.

torch is used for device memory and streams; no arithmetic of the method is
done here.  If the shared library is missing the import of the symbols fails
with an error that says how to build it -- there is no fallback path.
"""
from __future__ import annotations

import ctypes as C
import os
from dataclasses import dataclass

HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(HERE, "libkeyformer.so")

F32, BF16, F16 = 0, 1, 2
NOISE_NONE, NOISE_GUMBEL, NOISE_GAUSSIAN, NOISE_CONSTANT = 0, 1, 2, 3
LAYOUT_ORDERED, LAYOUT_SLOT = 0, 1
POS_ORIGINAL, POS_NEW = 0, 1
SCORE_PER_LAYER, SCORE_SHARED = 0, 1
KF_OK, KF_EINVAL, KF_EUNSUPPORTED, KF_EWORKSPACE, KF_EDEVICE = 0, -1, -2, -3, -4

# every symbol include/keyformer.h declares
SYMBOLS = ("kf_version", "kf_last_error", "kf_tau", "kf_noise_bits", "kf_workspace_bytes",
           "kf_prefill_score", "kf_decode_step", "kf_select_evict", "kf_select_evict_into", "kf_decode_select_step",
           "kf_decode_launch_shape", "kf_decode_select_step_at", "kf_beam_fork", "kf_decode_select_step_noalloc")
NOALLOC_SCRATCH_BYTES = 32 << 20


class KeyformerError(RuntimeError):
    def __init__(self, status, text):
        super().__init__("keyformer status %d: %s" % (status, text))
        self.status = status


class kf_cache(C.Structure):
    _fields_ = [("K", C.c_void_p), ("V", C.c_void_p), ("score", C.c_void_p), ("pos", C.c_void_p),
                ("len", C.c_void_p), ("L", C.c_int32), ("B", C.c_int32), ("H", C.c_int32),
                ("d", C.c_int32), ("cap", C.c_int32), ("dtype", C.c_int32), ("layer0", C.c_int32),
                ("q_per_kv", C.c_int32)]


class kf_score_cfg(C.Structure):
    _fields_ = [("tau", C.c_float), ("scale", C.c_float), ("noise", C.c_int32),
                ("seeds", C.c_void_p), ("alibi_slopes", C.c_void_p), ("pos_mode", C.c_int32),
                ("score_mode", C.c_int32), ("seq_q_pos", C.c_void_p), ("seq_tau", C.c_void_p),
                ("seq_n", C.c_void_p)]


class kf_schedule(C.Structure):
    _fields_ = [("n", C.c_int32), ("T", C.c_int32), ("tau_init", C.c_float), ("tau_end", C.c_float)]


_lib = None


def lib_path() -> str:
    return _LIB_PATH


def lib():
    """The loaded library.  Raises if it has not been built (no fallback)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise ImportError(
                "libkeyformer.so is not built: run `python -m paper_2403_09054_amd.build` "
                "(or __graft_entry__.build()) first; there is no CPU fallback")
        L = C.CDLL(_LIB_PATH)
        vp = C.c_void_p
        L.kf_version.restype = C.c_int32
        L.kf_version.argtypes = []
        L.kf_last_error.restype = C.c_char_p
        L.kf_last_error.argtypes = []
        L.kf_tau.restype = C.c_float
        L.kf_tau.argtypes = [C.c_int32, C.c_int32, C.c_float, C.c_float]
        L.kf_noise_bits.restype = C.c_uint32
        L.kf_noise_bits.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32]
        L.kf_workspace_bytes.restype = C.c_size_t
        L.kf_workspace_bytes.argtypes = [C.POINTER(kf_cache), C.c_int32]
        L.kf_decode_launch_shape.restype = C.c_int
        L.kf_decode_launch_shape.argtypes = [C.POINTER(kf_cache), C.c_int32, C.POINTER(C.c_int32),
                                             C.POINTER(C.c_int32)]
        L.kf_prefill_score.restype = C.c_int
        L.kf_prefill_score.argtypes = [C.POINTER(kf_cache), vp, C.c_int32, C.POINTER(kf_score_cfg), vp,
                                       C.c_size_t, vp]
        L.kf_decode_step.restype = C.c_int
        L.kf_decode_step.argtypes = [C.POINTER(kf_cache), vp, vp, vp, C.c_int32, C.c_int32,
                                     C.POINTER(kf_score_cfg), vp, vp, C.c_size_t, vp]
        L.kf_select_evict.restype = C.c_int
        L.kf_select_evict.argtypes = [C.POINTER(kf_cache), C.c_int32, C.c_int32, C.c_int32, vp, vp, C.c_size_t, vp]
        L.kf_select_evict_into.restype = C.c_int
        L.kf_select_evict_into.argtypes = [C.POINTER(kf_cache), C.POINTER(kf_cache), C.c_int32, C.c_int32, C.c_int32,
                                           vp, vp, C.c_size_t, vp]
        L.kf_beam_fork.restype = C.c_int
        L.kf_beam_fork.argtypes = [C.POINTER(kf_cache), vp, vp, C.c_size_t, vp]
        L.kf_decode_select_step.restype = C.c_int
        L.kf_decode_select_step.argtypes = [C.POINTER(kf_cache), vp, vp, vp, C.c_int32, C.c_int32,
                                            C.POINTER(kf_score_cfg), vp, C.c_int32, C.c_int32, C.c_int32, vp, vp,
                                            C.c_size_t, vp]
        L.kf_decode_select_step_at.restype = C.c_int
        L.kf_decode_select_step_at.argtypes = [C.POINTER(kf_cache), vp, vp, vp, C.POINTER(kf_schedule), vp, C.c_int32,
                                               C.POINTER(kf_score_cfg), vp, C.c_int32, C.c_int32, C.c_int32, vp, vp,
                                               C.c_size_t, vp]
        L.kf_decode_select_step_noalloc.restype = C.c_int
        L.kf_decode_select_step_noalloc.argtypes = [C.POINTER(kf_cache), vp, vp, vp, C.c_int32, C.c_int32,
                                                    C.POINTER(kf_score_cfg), vp, C.c_int32, C.c_int32, C.c_int32, vp,
                                                    vp, vp]
        _lib = L
    return _lib


def _check(rc):
    if rc != KF_OK:
        raise KeyformerError(rc, lib().kf_last_error().decode())


def kf_version() -> int:
    return int(lib().kf_version())


def kf_tau(t: int, T: int, tau_init: float = 1.0, tau_end: float = 2.0) -> float:
    return float(lib().kf_tau(t, T, tau_init, tau_end))


def kf_noise_bits(seed: int, layer: int, head: int, q_pos: int, k_pos: int) -> int:
    return int(lib().kf_noise_bits(seed, layer, head, q_pos, k_pos))


def _ptr(t):
    """Device (or fake, for host-only validation tests) address of a tensor / int / None."""
    return t if t is None or isinstance(t, int) else t.data_ptr()


@dataclass
class Cache:
    """Torch tensors that back a kf_cache.  K, V: [L,B,H,cap,d] (float32, bfloat16 or
    float16); score [L,B,H,cap] float32; pos [L,B,H,cap] int32; len [L,B,H] int32."""
    K: object
    V: object
    score: object
    pos: object
    len: object
    L: int
    B: int
    H: int
    d: int
    cap: int
    dtype: int
    layer0: int = 0
    q_per_kv: int = 1      # query heads served by each cached head (grouped-query attention if > 1)

    @staticmethod
    def allocate(L, B, H, d, cap, dtype=BF16, device="cuda", layer0=0, q_per_kv=1):
        import torch
        et = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16}[dtype]
        return Cache(K=torch.zeros((L, B, H, cap, d), dtype=et, device=device),
                     V=torch.zeros((L, B, H, cap, d), dtype=et, device=device),
                     score=torch.zeros((L, B, H, cap), dtype=torch.float32, device=device),
                     pos=torch.zeros((L, B, H, cap), dtype=torch.int32, device=device),
                     len=torch.zeros((L, B, H), dtype=torch.int32, device=device),
                     L=L, B=B, H=H, d=d, cap=cap, dtype=dtype, layer0=layer0, q_per_kv=q_per_kv)

    def c_struct(self) -> kf_cache:
        K, V, score, pos, lens = self.K, self.V, self.score, self.pos, self.len
        try:  # tensors, as in every call of a generation: without a choice for each
            K, V, score, pos, lens = K.data_ptr(), V.data_ptr(), score.data_ptr(), pos.data_ptr(), lens.data_ptr()
        except AttributeError:
            K, V, score, pos, lens = _ptr(K), _ptr(V), _ptr(score), _ptr(pos), _ptr(lens)
        return kf_cache(K, V, score, pos, lens, self.L, self.B, self.H, self.d, self.cap, self.dtype, self.layer0, self.q_per_kv)


def kf_workspace_bytes(cache: Cache, n_max: int = 0) -> int:
    cs = cache.c_struct()
    return int(lib().kf_workspace_bytes(C.byref(cs), n_max))


def kf_decode_launch_shape(cache: Cache, m_hint: int = 0):
    """(splits per unit, cache rows per split) of the decode launch for this cache."""
    cs = cache.c_struct()
    S, chunk = C.c_int32(0), C.c_int32(0)
    _check(lib().kf_decode_launch_shape(C.byref(cs), m_hint, C.byref(S), C.byref(chunk)))
    return S.value, chunk.value


def new_workspace(cache: Cache, n_max: int = 0, device="cuda"):
    """A zero-filled workspace tensor large enough for every call on `cache`."""
    import torch
    nbytes = kf_workspace_bytes(cache, n_max)
    if nbytes == 0:
        raise KeyformerError(KF_EUNSUPPORTED, "unsupported cache shape")
    return torch.zeros((nbytes + 15) // 16 * 16, dtype=torch.uint8, device=device)


def _stream(stream):
    """Handle of the stream a call goes to.  The smallest calls are bound by their host work; asking whether there is a GPU
    and for a stream object was a fifth of it (1 x 2 heads x 64 x 64, with the cache's addresses read in one go: 15.4 ->
    12.5 us a step), and is left out once torch runs on a GPU."""
    if stream is None:
        import torch
        if torch.cuda.is_initialized():
            try:
                return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
            except AttributeError:  # a torch without these two: by way of its stream object
                pass
        return torch.cuda.current_stream().cuda_stream if torch.cuda.is_available() else None
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _ws(workspace):
    if workspace is None:
        return None, 0
    if isinstance(workspace, tuple):  # (address, bytes), for host-only tests
        return workspace
    return workspace.data_ptr(), workspace.numel() * workspace.element_size()


def _cfg(tau, scale, noise, seeds, slopes, pos_mode=0, score_mode=0, seq_q_pos=None, seq_tau=None,
         seq_n=None) -> kf_score_cfg:
    return kf_score_cfg(tau, scale, noise, _ptr(seeds), _ptr(slopes), pos_mode, score_mode, _ptr(seq_q_pos),
                        _ptr(seq_tau), _ptr(seq_n))


def kf_prefill_score(cache: Cache, Q, n: int, tau: float, scale: float, noise: int = NOISE_GUMBEL,
                     seeds=None, slopes=None, workspace=None, stream=None,
                     score_mode: int = SCORE_PER_LAYER, seq_n=None) -> None:
    """seq_n: int32 device tensor [B] of per-sequence prompt lengths (prompts padded to n), or None."""
    cs, cfg = cache.c_struct(), _cfg(tau, scale, noise, seeds, slopes, 0, score_mode, seq_n=seq_n)
    wp, wb = _ws(workspace)
    _check(lib().kf_prefill_score(C.byref(cs), _ptr(Q), n, C.byref(cfg), wp, wb, _stream(stream)))


def kf_beam_fork(cache: Cache, parent, workspace=None, stream=None) -> None:
    """parent: int32 device tensor [B]; row b of the batch takes over the cache state of row parent[b]."""
    cs = cache.c_struct()
    wp, wb = _ws(workspace)
    _check(lib().kf_beam_fork(C.byref(cs), _ptr(parent), wp, wb, _stream(stream)))


def kf_decode_step(cache: Cache, q, k_new, v_new, q_pos: int, m_hint: int, tau: float, scale: float,
                   noise: int = NOISE_GUMBEL, seeds=None, slopes=None, out=None, workspace=None,
                   stream=None, pos_mode: int = POS_ORIGINAL, score_mode: int = SCORE_PER_LAYER,
                   seq_q_pos=None, seq_tau=None) -> None:
    cs, cfg = cache.c_struct(), _cfg(tau, scale, noise, seeds, slopes, pos_mode, score_mode, seq_q_pos, seq_tau)
    wp, wb = _ws(workspace)
    _check(lib().kf_decode_step(C.byref(cs), _ptr(q), _ptr(k_new), _ptr(v_new), q_pos, m_hint,
                                C.byref(cfg), _ptr(out), wp, wb, _stream(stream)))


def kf_select_evict(cache: Cache, k: int, w: int, kept_idx=None, workspace=None, stream=None,
                    layout: int = LAYOUT_ORDERED) -> None:
    cs = cache.c_struct()
    wp, wb = _ws(workspace)
    _check(lib().kf_select_evict(C.byref(cs), k, w, layout, _ptr(kept_idx), wp, wb, _stream(stream)))


def kf_select_evict_into(src: Cache, dst: Cache, dst_layer0: int, k: int, w: int, kept_idx=None, workspace=None,
                         stream=None) -> None:
    ss, ds = src.c_struct(), dst.c_struct()
    wp, wb = _ws(workspace)
    _check(lib().kf_select_evict_into(C.byref(ss), C.byref(ds), dst_layer0, k, w, _ptr(kept_idx), wp, wb,
                                      _stream(stream)))


def kf_decode_select_step(cache: Cache, q, k_new, v_new, q_pos: int, m_hint: int, tau: float, scale: float,
                          noise: int = NOISE_GUMBEL, seeds=None, slopes=None, out=None, k: int = 0, w: int = 0,
                          layout: int = LAYOUT_ORDERED, kept_idx=None, workspace=None, stream=None,
                          pos_mode: int = POS_ORIGINAL, score_mode: int = SCORE_PER_LAYER,
                          seq_q_pos=None, seq_tau=None) -> None:
    cs, cfg = cache.c_struct(), _cfg(tau, scale, noise, seeds, slopes, pos_mode, score_mode, seq_q_pos, seq_tau)
    wp, wb = _ws(workspace)
    _check(lib().kf_decode_select_step(C.byref(cs), _ptr(q), _ptr(k_new), _ptr(v_new), q_pos, m_hint,
                                       C.byref(cfg), _ptr(out), k, w, layout, _ptr(kept_idx), wp, wb,
                                       _stream(stream)))


def kf_decode_select_step_at(cache: Cache, q, k_new, v_new, n: int, T: int, tau_init: float, tau_end: float, step,
                             m_hint: int, scale: float, noise: int = NOISE_GUMBEL, seeds=None, slopes=None,
                             out=None, k: int = 0, w: int = 0, layout: int = LAYOUT_ORDERED, kept_idx=None,
                             workspace=None, stream=None, pos_mode: int = POS_ORIGINAL,
                             score_mode: int = SCORE_PER_LAYER) -> None:
    """`step`: int32 device tensor of one element holding the decode step number."""
    cs, cfg = cache.c_struct(), _cfg(1.0, scale, noise, seeds, slopes, pos_mode, score_mode)
    sched = kf_schedule(n, T, tau_init, tau_end)
    wp, wb = _ws(workspace)
    _check(lib().kf_decode_select_step_at(C.byref(cs), _ptr(q), _ptr(k_new), _ptr(v_new), C.byref(sched),
                                          _ptr(step), m_hint, C.byref(cfg), _ptr(out), k, w, layout,
                                          _ptr(kept_idx), wp, wb, _stream(stream)))


def kf_decode_select_step_noalloc(cache: Cache, q, k_new, v_new, q_pos: int, m_hint: int, tau: float, scale: float,
                                  noise: int = NOISE_GUMBEL, seeds=None, slopes=None, out=None, k: int = 0, w: int = 0,
                                  layout: int = LAYOUT_ORDERED, kept_idx=None, skipped=None, stream=None,
                                  pos_mode: int = POS_ORIGINAL, score_mode: int = SCORE_PER_LAYER,
                                  seq_q_pos=None, seq_tau=None) -> None:
    """kf_decode_select_step on the library's built-in scratch (no workspace argument).  `skipped`: int32
    device tensor of one element that counts skipped units, or None."""
    cs, cfg = cache.c_struct(), _cfg(tau, scale, noise, seeds, slopes, pos_mode, score_mode, seq_q_pos, seq_tau)
    _check(lib().kf_decode_select_step_noalloc(C.byref(cs), _ptr(q), _ptr(k_new), _ptr(v_new), q_pos, m_hint,
                                               C.byref(cfg), _ptr(out), k, w, layout, _ptr(kept_idx),
                                               _ptr(skipped), _stream(stream)))
