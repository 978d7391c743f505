"""ctypes binding of libimpact.so: argument marshalling only.

Every function here has the name of the C entry point it calls (``include/impact.h``)
and passes raw device pointers taken from torch tensors.  No arithmetic of the loss
or of the buffer happens in Python.
"""
from __future__ import annotations

import ctypes
import math
import os
from dataclasses import dataclass
from typing import Dict, Optional, Tuple

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# IMPACT_LIB_PATH: load this build of the library instead (e.g. one compiled with sanitizers)
LIB_PATH = os.environ.get("IMPACT_LIB_PATH") or os.path.join(_HERE, "libimpact.so")

IMPACT_OK = 0
IMPACT_ERR_INVALID_ARG = -1
IMPACT_ERR_BUFFER_FULL = -2
IMPACT_ERR_NOT_ENOUGH_LIVE = -3
IMPACT_ERR_HIP = -4
IMPACT_ERR_UNSUPPORTED = -5
IMPACT_ERR_TOO_LARGE = -6
IMPACT_STATIC_WORKSPACE_BYTES = 2 << 20

IMPACT_CATEGORICAL = 0
IMPACT_DIAG_GAUSSIAN = 1
IMPACT_F32 = 0
IMPACT_BF16 = 1
IMPACT_FLAG_FORCE_GENERIC = 1
IMPACT_FLAG_RATIO_WORKER = 2
IMPACT_FLAG_LEARNER_BF16 = 4
IMPACT_FLAG_BATCH_MAJOR = 8
IMPACT_FLAG_ACTIONS_U8 = 16
IMPACT_LANES = 16


def IMPACT_FLAG_LANE(n: int) -> int:
    return (n & 15) << 8

IMPACT_BUFFER_CACHE_LOGP = 1
IMPACT_BUFFER_NO_TARGET_DIST = 2
IMPACT_BUFFER_ACTIONS_U8 = 4

EXPORTS = [
    "impact_version", "impact_status_string",
    "impact_buffer_storage_bytes", "impact_buffer_create", "impact_buffer_destroy", "impact_buffer_num_live",
    "impact_buffer_num_empty", "impact_buffer_release_discarded", "impact_buffer_missing_targets",
    "impact_buffer_mark_target", "impact_buffer_learner_step", "impact_target_period", "impact_buffer_reset_lanes",
    "impact_buffer_state_bytes", "impact_buffer_export_state", "impact_buffer_import_state",
    "impact_buffer_reserve", "impact_buffer_insert", "impact_buffer_put_target", "impact_buffer_sample",
    "impact_buffer_gather", "impact_loss_workspace_bytes", "impact_loss_fwd_bwd",
    "impact_loss_fwd_bwd_from_buffer", "impact_loss_fwd_bwd_static",
]


class ImpactError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: status {status} ({status_string(status)})")


class impact_buffer_desc_t(ctypes.Structure):
    _fields_ = [("dist", ctypes.c_int32), ("T", ctypes.c_int32), ("A", ctypes.c_int32),
                ("num_slots", ctypes.c_int32), ("K", ctypes.c_int32), ("storage", ctypes.c_int32),
                ("flags", ctypes.c_uint32)]


class impact_loss_config_t(ctypes.Structure):
    _fields_ = [("gamma", ctypes.c_float), ("lam", ctypes.c_float), ("rho_bar", ctypes.c_float),
                ("c_bar", ctypes.c_float), ("rho_clip", ctypes.c_float), ("eps", ctypes.c_float),
                ("vf_coeff", ctypes.c_float), ("ent_coeff", ctypes.c_float), ("kl_coeff", ctypes.c_float),
                ("flags", ctypes.c_uint32)]


class impact_batch_t(ctypes.Structure):
    _fields_ = [("worker_dist", ctypes.c_void_p), ("target_dist", ctypes.c_void_p), ("actions", ctypes.c_void_p),
                ("rewards", ctypes.c_void_p), ("dones", ctypes.c_void_p), ("logp", ctypes.c_void_p)]


class impact_loss_out_t(ctypes.Structure):
    _fields_ = [("grad_learner_dist", ctypes.c_void_p), ("grad_values", ctypes.c_void_p), ("vs", ctypes.c_void_p),
                ("adv", ctypes.c_void_p), ("loss5", ctypes.c_void_p), ("step_outputs", ctypes.c_void_p),
                ("fractions", ctypes.c_void_p)]


_lib: Optional[ctypes.CDLL] = None


def load() -> ctypes.CDLL:
    """Load libimpact.so.  There is no fallback: a missing library is an error."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise ImportError(f"{LIB_PATH} is missing: build it with `python -m paper_1912_00167_amd.build`")
    L = ctypes.CDLL(LIB_PATH)
    vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    L.impact_version.restype = ctypes.c_char_p
    L.impact_status_string.restype = ctypes.c_char_p
    L.impact_status_string.argtypes = [ctypes.c_int]
    L.impact_buffer_storage_bytes.restype = sz
    L.impact_buffer_storage_bytes.argtypes = [ctypes.POINTER(impact_buffer_desc_t)]
    L.impact_buffer_create.restype = ctypes.c_int
    L.impact_buffer_create.argtypes = [ctypes.POINTER(impact_buffer_desc_t), vp, sz, ctypes.POINTER(vp)]
    L.impact_buffer_destroy.restype = ctypes.c_int
    L.impact_buffer_destroy.argtypes = [vp]
    L.impact_buffer_num_live.restype = i32
    L.impact_buffer_num_live.argtypes = [vp]
    L.impact_buffer_num_empty.restype = i32
    L.impact_buffer_num_empty.argtypes = [vp]
    L.impact_buffer_release_discarded.restype = ctypes.c_int
    L.impact_buffer_release_discarded.argtypes = [vp]
    L.impact_buffer_missing_targets.restype = ctypes.c_int
    L.impact_buffer_missing_targets.argtypes = [vp, i32, vp, vp, vp]
    L.impact_buffer_mark_target.restype = ctypes.c_int
    L.impact_buffer_mark_target.argtypes = [vp, i32, vp]
    L.impact_buffer_learner_step.restype = ctypes.c_int
    L.impact_buffer_learner_step.argtypes = [vp, ctypes.c_int64, vp, vp]
    L.impact_target_period.restype = ctypes.c_int64
    L.impact_target_period.argtypes = [i32, i32, i32]
    L.impact_buffer_reset_lanes.restype = ctypes.c_int
    L.impact_buffer_reset_lanes.argtypes = [vp]
    L.impact_buffer_state_bytes.restype = sz
    L.impact_buffer_state_bytes.argtypes = [vp]
    L.impact_buffer_export_state.restype = ctypes.c_int
    L.impact_buffer_export_state.argtypes = [vp, vp, sz]
    L.impact_buffer_import_state.restype = ctypes.c_int
    L.impact_buffer_import_state.argtypes = [vp, vp, sz]
    L.impact_buffer_reserve.restype = ctypes.c_int
    L.impact_buffer_reserve.argtypes = [vp, i32, vp]
    L.impact_buffer_insert.restype = ctypes.c_int
    L.impact_buffer_insert.argtypes = [vp, i32, ctypes.POINTER(impact_batch_t), vp, vp]
    L.impact_buffer_put_target.restype = ctypes.c_int
    L.impact_buffer_put_target.argtypes = [vp, i32, vp, vp, vp]
    L.impact_buffer_sample.restype = ctypes.c_int
    L.impact_buffer_sample.argtypes = [vp, i32, vp, vp]
    L.impact_buffer_gather.restype = ctypes.c_int
    L.impact_buffer_gather.argtypes = [vp, i32, vp, ctypes.POINTER(impact_batch_t), vp]
    L.impact_loss_workspace_bytes.restype = sz
    L.impact_loss_workspace_bytes.argtypes = [i32, i32, i32, i32]
    L.impact_loss_fwd_bwd.restype = ctypes.c_int
    L.impact_loss_fwd_bwd.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, ctypes.POINTER(impact_batch_t),
                                      ctypes.POINTER(impact_loss_config_t), ctypes.POINTER(impact_loss_out_t),
                                      vp, sz, vp]
    L.impact_loss_fwd_bwd_from_buffer.restype = ctypes.c_int
    L.impact_loss_fwd_bwd_from_buffer.argtypes = [vp, i32, vp, vp, vp, vp, ctypes.POINTER(impact_loss_config_t),
                                                  ctypes.POINTER(impact_loss_out_t), vp, sz, vp]
    L.impact_loss_fwd_bwd_static.restype = ctypes.c_int
    L.impact_loss_fwd_bwd_static.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, ctypes.POINTER(impact_batch_t),
                                             ctypes.POINTER(impact_loss_config_t), ctypes.POINTER(impact_loss_out_t), vp]
    _lib = L
    return L


def impact_version() -> str:
    return load().impact_version().decode()


def status_string(status: int) -> str:
    return load().impact_status_string(int(status)).decode()


def _check(status: int, where: str) -> None:
    if status != IMPACT_OK:
        raise ImpactError(status, where)


# Addresses go to the library as plain integers, which ctypes converts by the functions' declared argument types: a small
# call's time on the host is that of the objects made on the way (17 -> 12 us per sample + loss).

def _ptr(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not t.is_contiguous():
        raise ValueError("tensors handed to libimpact must be contiguous")
    return t.data_ptr()


def _expect(name: str, t: Optional[torch.Tensor], dtype, shape, optional: bool = False) -> None:
    """The C side sees addresses only: a tensor of another element type or shape than the call reads or
    writes would send a kernel outside the allocation, so that is refused here."""
    if t is None:
        if optional:
            return
        raise ValueError(f"{name}: missing")
    if t.dtype is not dtype and (not isinstance(dtype, tuple) or t.dtype not in dtype):
        want = " or ".join(str(d) for d in dtype) if isinstance(dtype, tuple) else str(dtype)
        raise TypeError(f"{name}: expected {want}, got {t.dtype}")
    if t.shape != shape:                               # (torch.Size compares equal to a tuple of the same numbers)
        raise ValueError(f"{name}: expected shape {tuple(shape)}, got {tuple(t.shape)}")


def _stream(stream) -> int:
    if stream is None:
        if torch.cuda.is_initialized():            # the handle alone, without an object around it
            return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
        stream = torch.cuda.current_stream()
    return stream.cuda_stream


def dist_code(dist) -> int:
    return {"categorical": IMPACT_CATEGORICAL, "gaussian": IMPACT_DIAG_GAUSSIAN,
            IMPACT_CATEGORICAL: IMPACT_CATEGORICAL, IMPACT_DIAG_GAUSSIAN: IMPACT_DIAG_GAUSSIAN}[dist]


def dtype_code(storage) -> int:
    return {"f32": IMPACT_F32, "bf16": IMPACT_BF16, IMPACT_F32: IMPACT_F32, IMPACT_BF16: IMPACT_BF16,
            torch.float32: IMPACT_F32, torch.bfloat16: IMPACT_BF16}[storage]


def make_config(gamma=0.99, lam=1.0, rho_bar=1.0, c_bar=1.0, rho_clip=2.0, eps=0.2, vf_coeff=1.0,
                ent_coeff=0.01, kl_coeff=0.0, flags=0) -> impact_loss_config_t:
    return impact_loss_config_t(gamma, lam, rho_bar, c_bar, rho_clip, eps, vf_coeff, ent_coeff, kl_coeff, flags)


def config_from_hyper(h, flags: int = 0) -> impact_loss_config_t:
    if getattr(h, "ratio_mode", 0) == 1:
        flags |= IMPACT_FLAG_RATIO_WORKER
    return make_config(h.gamma, h.lam, h.rho_bar, h.c_bar, h.rho_clip, h.eps, h.vf_coeff, h.ent_coeff,
                       h.kl_coeff, flags)


def _cfg_for(cfg: impact_loss_config_t, learner: torch.Tensor) -> impact_loss_config_t:
    """The configuration with the learner tensor's dtype flagged (fp32 or bf16)."""
    if learner.dtype == torch.float32:
        return cfg
    if learner.dtype != torch.bfloat16:
        raise ValueError("the learner's distribution tensor is fp32 or bf16")
    c = impact_loss_config_t.from_buffer_copy(cfg)
    c.flags |= IMPACT_FLAG_LEARNER_BF16
    return c


def _batch_struct(batch: Dict[str, torch.Tensor], need_target: bool = True) -> impact_batch_t:
    """worker/target may be missing where cached log-probabilities ("logp", fp64 [T][B][2]) stand in for them."""
    tgt, lp = batch.get("target"), batch.get("logp")
    if need_target and tgt is None and lp is None:
        raise ValueError("batch needs a target tensor")
    if lp is not None and lp.dtype != torch.float64:
        raise ValueError("cached log-probabilities are fp64")
    return impact_batch_t(_ptr(batch.get("worker")), _ptr(tgt), _ptr(batch["actions"]), _ptr(batch["rewards"]),
                          _ptr(batch["dones"]), _ptr(lp))


# ------------------------------------------------------------------------------------------
# circular buffer
# ------------------------------------------------------------------------------------------

def impact_buffer_storage_bytes(dist, T: int, A: int, num_slots: int, K: int, storage, flags: int = 0) -> int:
    d = impact_buffer_desc_t(dist_code(dist), T, A, num_slots, K, dtype_code(storage), flags)
    return int(load().impact_buffer_storage_bytes(ctypes.byref(d)))


class Buffer:
    """Owner of a buffer handle and of the torch allocation behind it."""

    def __init__(self, dist, T: int, A: int, num_slots: int, K: int, storage="f32", device="cuda", flags: int = 0):
        self.desc = impact_buffer_desc_t(dist_code(dist), T, A, num_slots, K, dtype_code(storage), flags)
        self.flags = flags
        nbytes = int(load().impact_buffer_storage_bytes(ctypes.byref(self.desc)))
        if nbytes == 0:
            raise ImpactError(IMPACT_ERR_INVALID_ARG, "impact_buffer_storage_bytes")
        # (the library wants its storage on a 256-byte boundary; device allocations are, host ones may not be)
        self._raw = torch.zeros(nbytes + 255, dtype=torch.uint8, device=device)
        skip = -self._raw.data_ptr() % 256
        self.storage = self._raw[skip: skip + nbytes]
        self.handle = ctypes.c_void_p()
        _check(load().impact_buffer_create(ctypes.byref(self.desc), _ptr(self.storage), nbytes,
                                           ctypes.byref(self.handle)), "impact_buffer_create")
        self.dist, self.T, self.A, self.num_slots, self.K = self.desc.dist, T, A, num_slots, K
        self.W = A if self.dist == IMPACT_CATEGORICAL else 2 * A
        self.float_dtype = torch.float32 if self.desc.storage == IMPACT_F32 else torch.bfloat16
        # what `actions` of insert and gather holds
        self.action_dtype = (self.float_dtype if self.dist != IMPACT_CATEGORICAL
                             else torch.uint8 if flags & IMPACT_BUFFER_ACTIONS_U8 else torch.int32)
        self.device = self.storage.device

    def close(self) -> None:
        if self.handle:
            load().impact_buffer_destroy(self.handle)
            self.handle = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def impact_buffer_num_live(buf: Buffer) -> int:
    return int(load().impact_buffer_num_live(buf.handle))


def impact_buffer_num_empty(buf: Buffer) -> int:
    return int(load().impact_buffer_num_empty(buf.handle))


def impact_buffer_release_discarded(buf: Buffer) -> None:
    _check(load().impact_buffer_release_discarded(buf.handle), "impact_buffer_release_discarded")


def impact_buffer_missing_targets(buf: Buffer, slots: np.ndarray) -> np.ndarray:
    """Positions in the batch whose slot holds no target output yet."""
    slots = np.ascontiguousarray(slots, dtype=np.int32)
    pos = np.empty(max(slots.size, 1), dtype=np.int32)
    n = ctypes.c_int32(0)
    _check(load().impact_buffer_missing_targets(buf.handle, slots.size, slots.ctypes.data,
                                                pos.ctypes.data, ctypes.byref(n)),
           "impact_buffer_missing_targets")
    return pos[: n.value].copy()


def impact_buffer_mark_target(buf: Buffer, slots: np.ndarray) -> None:
    slots = np.ascontiguousarray(slots, dtype=np.int32)
    _check(load().impact_buffer_mark_target(buf.handle, slots.size, slots.ctypes.data),
           "impact_buffer_mark_target")


def impact_buffer_learner_step(buf: Buffer, t_target: int) -> Tuple[int, bool]:
    """Counts one learner step; returns (t, target update due)."""
    t, due = ctypes.c_int64(0), ctypes.c_int32(0)
    _check(load().impact_buffer_learner_step(buf.handle, int(t_target), ctypes.byref(t), ctypes.byref(due)),
           "impact_buffer_learner_step")
    return int(t.value), bool(due.value)


def impact_target_period(num_slots: int, B: int, K: int) -> int:
    return int(load().impact_target_period(num_slots, B, K))


def impact_buffer_reset_lanes(buf: Buffer) -> None:
    _check(load().impact_buffer_reset_lanes(buf.handle), "impact_buffer_reset_lanes")


def impact_buffer_export_state(buf: Buffer) -> np.ndarray:
    """The ring's bookkeeping as a byte array (the slots' contents stay in the caller's device storage)."""
    L = load()
    state = np.empty(int(L.impact_buffer_state_bytes(buf.handle)), dtype=np.uint8)
    _check(L.impact_buffer_export_state(buf.handle, state.ctypes.data, state.size),
           "impact_buffer_export_state")
    return state


def impact_buffer_import_state(buf: Buffer, state: np.ndarray) -> None:
    state = np.ascontiguousarray(state, dtype=np.uint8)
    _check(load().impact_buffer_import_state(buf.handle, state.ctypes.data, state.size),
           "impact_buffer_import_state")


def impact_buffer_reserve(buf: Buffer, n: int) -> np.ndarray:
    slots = np.empty(max(n, 0), dtype=np.int32)
    _check(load().impact_buffer_reserve(buf.handle, n, slots.ctypes.data), "impact_buffer_reserve")
    return slots


def impact_buffer_insert(buf: Buffer, src: Dict[str, torch.Tensor], stream=None) -> np.ndarray:
    """src: time-major fp32 device tensors worker/actions/rewards/dones (+ optional target)."""
    n = int(src["worker"].shape[1])
    T, f32 = buf.T, torch.float32
    _expect("worker", src.get("worker"), f32, (T, n, buf.W))
    _expect("target", src.get("target"), f32, (T, n, buf.W), optional=True)
    if buf.dist == IMPACT_CATEGORICAL:
        _expect("actions", src.get("actions"), buf.action_dtype, (T, n))
    else:
        _expect("actions", src.get("actions"), f32, (T, n, buf.A))
    _expect("rewards", src.get("rewards"), f32, (T, n))
    _expect("dones", src.get("dones"), torch.uint8, (T, n))
    slots = np.empty(n, dtype=np.int32)
    b = _batch_struct(src, need_target=False)
    _check(load().impact_buffer_insert(buf.handle, n, ctypes.byref(b), slots.ctypes.data,
                                       _stream(stream)), "impact_buffer_insert")
    return slots


def impact_buffer_put_target(buf: Buffer, slots: np.ndarray, target: torch.Tensor, stream=None) -> None:
    slots = np.ascontiguousarray(slots, dtype=np.int32)
    _expect("target", target, torch.float32, (buf.T, slots.size, buf.W))
    _check(load().impact_buffer_put_target(buf.handle, slots.size, slots.ctypes.data,
                                           _ptr(target), _stream(stream)), "impact_buffer_put_target")


def impact_buffer_sample(buf: Buffer, B: int, out_slots: Optional[np.ndarray] = None,
                         out_counts: Optional[np.ndarray] = None) -> Tuple[np.ndarray, np.ndarray]:
    if out_slots is None:
        out_slots = np.empty(max(B, 0), dtype=np.int32)
    if out_counts is None:
        out_counts = np.empty(max(B, 0), dtype=np.int32)
    _check(load().impact_buffer_sample(buf.handle, B, out_slots.ctypes.data,
                                       out_counts.ctypes.data), "impact_buffer_sample")
    return out_slots, out_counts


def alloc_batch(buf: Buffer, B: int) -> Dict[str, torch.Tensor]:
    """Device tensors able to receive a gathered batch (storage dtype)."""
    fd, dev, T = buf.float_dtype, buf.device, buf.T
    acts = (torch.empty((T, B), dtype=buf.action_dtype, device=dev) if buf.dist == IMPACT_CATEGORICAL
            else torch.empty((T, B, buf.A), dtype=fd, device=dev))
    out = dict(actions=acts, rewards=torch.empty((T, B), dtype=fd, device=dev),
               dones=torch.empty((T, B), dtype=torch.uint8, device=dev))
    if buf.flags & IMPACT_BUFFER_CACHE_LOGP:
        out["logp"] = torch.empty((T, B, 2), dtype=torch.float64, device=dev)
    else:
        out["worker"] = torch.empty((T, B, buf.W), dtype=fd, device=dev)
    if not buf.flags & IMPACT_BUFFER_NO_TARGET_DIST:
        out["target"] = torch.empty((T, B, buf.W), dtype=fd, device=dev)
    return out


def _expect_batch(dist: int, fdt, idt, T: int, B: int, A: int, batch: Dict[str, torch.Tensor], gather_from=None) -> None:
    """Element types and shapes of the buffer-resident part of a time-major batch (fdt: its float type; idt: the
    type of a categorical action index).  gather_from: the buffer whose planes a gather fills it from."""
    W = A if dist == IMPACT_CATEGORICAL else 2 * A
    if gather_from is not None:
        need_worker = not gather_from.flags & IMPACT_BUFFER_CACHE_LOGP
        need_target = not gather_from.flags & IMPACT_BUFFER_NO_TARGET_DIST
        need_logp = bool(gather_from.flags & IMPACT_BUFFER_CACHE_LOGP)
    else:
        need_logp = batch.get("logp") is not None
        need_worker, need_target = not need_logp, not need_logp
    _expect("worker", batch.get("worker"), fdt, (T, B, W), optional=not need_worker)
    _expect("target", batch.get("target"), fdt, (T, B, W), optional=not need_target)
    _expect("logp", batch.get("logp"), torch.float64, (T, B, 2), optional=not need_logp)
    if dist == IMPACT_CATEGORICAL:
        _expect("actions", batch.get("actions"), idt, (T, B))
    else:
        _expect("actions", batch.get("actions"), fdt, (T, B, A))
    _expect("rewards", batch.get("rewards"), fdt, (T, B))
    _expect("dones", batch.get("dones"), torch.uint8, (T, B))


def _expect_learner_side(T: int, B: int, W: int, learner, values, bootstrap, cfg, out) -> None:
    bm = bool(cfg.flags & IMPACT_FLAG_BATCH_MAJOR)
    tb = (B, T) if bm else (T, B)
    _expect("learner", learner, (torch.float32, torch.bfloat16), tb + (W,))
    _expect("values", values, torch.float32, tb)
    _expect("bootstrap", bootstrap, torch.float32, (B,))
    f32 = torch.float32
    _expect("grad_dist", out.get("grad_dist"), f32, tb + (W,))
    _expect("loss5", out.get("loss5"), f32, (5,))
    _expect("fractions", out.get("fractions"), f32, (2,), optional=True)
    if out.get("step_outputs") is not None:
        _expect("step_outputs", out["step_outputs"], f32, tb + (4,))
    else:
        _expect("grad_values", out.get("grad_values"), f32, tb)
        _expect("vs", out.get("vs"), f32, tb, optional=True)
        _expect("adv", out.get("adv"), f32, tb, optional=True)


def impact_buffer_gather(buf: Buffer, dev_slots: torch.Tensor, dst: Optional[Dict[str, torch.Tensor]] = None,
                         stream=None) -> Dict[str, torch.Tensor]:
    B = int(dev_slots.numel())
    if dst is None:
        dst = alloc_batch(buf, B)
    _expect("slots", dev_slots, torch.int32, (B,))
    _expect_batch(buf.dist, buf.float_dtype, buf.action_dtype, buf.T, B, buf.A, dst, gather_from=buf)
    b = _batch_struct(dst)
    _check(load().impact_buffer_gather(buf.handle, B, _ptr(dev_slots), ctypes.byref(b), _stream(stream)),
           "impact_buffer_gather")
    return dst


# ------------------------------------------------------------------------------------------
# loss
# ------------------------------------------------------------------------------------------

def impact_loss_workspace_bytes(dist, T: int, B: int, A: int) -> int:
    return int(load().impact_loss_workspace_bytes(dist_code(dist), T, B, A))


def alloc_loss_out(T: int, B: int, W: int, device="cuda", want_targets: bool = True,
                   packed: bool = False) -> Dict[str, torch.Tensor]:
    """packed: the per-step scalars as one record {dL/dV, vs, adv, 0} per step ("step_outputs", [T][B][4]);
    grad_values, vs and adv are then strided views of it."""
    if packed:
        rec = torch.empty((T, B, 4), dtype=torch.float32, device=device)
        return dict(grad_dist=torch.empty((T, B, W), dtype=torch.float32, device=device), step_outputs=rec,
                    grad_values=rec[..., 0], vs=rec[..., 1], adv=rec[..., 2],
                    loss5=torch.empty(5, dtype=torch.float32, device=device),
                    fractions=torch.empty(2, dtype=torch.float32, device=device))
    out = dict(grad_dist=torch.empty((T, B, W), dtype=torch.float32, device=device),
               grad_values=torch.empty((T, B), dtype=torch.float32, device=device),
               loss5=torch.empty(5, dtype=torch.float32, device=device),
               fractions=torch.empty(2, dtype=torch.float32, device=device))
    if want_targets:
        out["vs"] = torch.empty((T, B), dtype=torch.float32, device=device)
        out["adv"] = torch.empty((T, B), dtype=torch.float32, device=device)
    return out


def _tbw(learner: torch.Tensor, cfg: impact_loss_config_t) -> Tuple[int, int, int]:
    """T, B, W from the learner tensor: [T][B][W], or [B][T][W] under IMPACT_FLAG_BATCH_MAJOR."""
    d0, d1, W = learner.shape
    return (d1, d0, W) if cfg.flags & IMPACT_FLAG_BATCH_MAJOR else (d0, d1, W)


def _out_struct(out: Dict[str, torch.Tensor]) -> impact_loss_out_t:
    if out.get("step_outputs") is not None:
        return impact_loss_out_t(_ptr(out["grad_dist"]), None, None, None, _ptr(out["loss5"]), _ptr(out["step_outputs"]),
                                 _ptr(out.get("fractions")))
    return impact_loss_out_t(_ptr(out["grad_dist"]), _ptr(out["grad_values"]), _ptr(out.get("vs")),
                             _ptr(out.get("adv")), _ptr(out["loss5"]), None, _ptr(out.get("fractions")))


def impact_loss_fwd_bwd(dist, learner: torch.Tensor, values: torch.Tensor, bootstrap: torch.Tensor,
                        batch: Dict[str, torch.Tensor], cfg: impact_loss_config_t,
                        out: Optional[Dict[str, torch.Tensor]] = None, workspace: Optional[torch.Tensor] = None,
                        stream=None) -> Dict[str, torch.Tensor]:
    d = dist_code(dist)
    T, B, W = _tbw(learner, cfg)
    A = W if d == IMPACT_CATEGORICAL else W // 2
    if out is None:
        out = alloc_loss_out(*((B, T, W) if cfg.flags & IMPACT_FLAG_BATCH_MAJOR else (T, B, W)), learner.device)
    if workspace is None:
        workspace = torch.empty(impact_loss_workspace_bytes(d, T, B, A), dtype=torch.uint8, device=learner.device)
    _expect_learner_side(T, B, W, learner, values, bootstrap, cfg, out)
    _expect_batch(d, batch["rewards"].dtype, torch.uint8 if cfg.flags & IMPACT_FLAG_ACTIONS_U8 else torch.int32, T, B, A, batch)
    b, o = _batch_struct(batch), _out_struct(out)
    cfg = _cfg_for(cfg, learner)
    _check(load().impact_loss_fwd_bwd(d, dtype_code(batch["rewards"].dtype), T, B, A, _ptr(learner), _ptr(values),
                                      _ptr(bootstrap), ctypes.byref(b), ctypes.byref(cfg), ctypes.byref(o),
                                      _ptr(workspace), workspace.numel(), _stream(stream)), "impact_loss_fwd_bwd")
    return out


def impact_loss_fwd_bwd_static(dist, learner: torch.Tensor, values: torch.Tensor, bootstrap: torch.Tensor,
                               batch: Dict[str, torch.Tensor], cfg: impact_loss_config_t,
                               out: Dict[str, torch.Tensor], stream=None) -> Dict[str, torch.Tensor]:
    """The caller brings every tensor (outputs included): this call allocates nothing, here or in the library."""
    d = dist_code(dist)
    T, B, W = _tbw(learner, cfg)
    A = W if d == IMPACT_CATEGORICAL else W // 2
    _expect_learner_side(T, B, W, learner, values, bootstrap, cfg, out)
    _expect_batch(d, batch["rewards"].dtype, torch.uint8 if cfg.flags & IMPACT_FLAG_ACTIONS_U8 else torch.int32, T, B, A, batch)
    b, o = _batch_struct(batch), _out_struct(out)
    cfg = _cfg_for(cfg, learner)
    _check(load().impact_loss_fwd_bwd_static(d, dtype_code(batch["rewards"].dtype), T, B, A, _ptr(learner), _ptr(values),
                                             _ptr(bootstrap), ctypes.byref(b), ctypes.byref(cfg), ctypes.byref(o),
                                             _stream(stream)), "impact_loss_fwd_bwd_static")
    return out


def impact_loss_fwd_bwd_from_buffer(buf: Buffer, dev_slots: torch.Tensor, learner: torch.Tensor,
                                    values: torch.Tensor, bootstrap: torch.Tensor, cfg: impact_loss_config_t,
                                    out: Optional[Dict[str, torch.Tensor]] = None,
                                    workspace: Optional[torch.Tensor] = None, stream=None) -> Dict[str, torch.Tensor]:
    T, B, W = _tbw(learner, cfg)
    if out is None:
        out = alloc_loss_out(*((B, T, W) if cfg.flags & IMPACT_FLAG_BATCH_MAJOR else (T, B, W)), learner.device)
    if workspace is None:
        workspace = torch.empty(impact_loss_workspace_bytes(buf.dist, T, B, buf.A), dtype=torch.uint8,
                                device=learner.device)
    if W != buf.W or T != buf.T:
        raise ValueError(f"learner: a buffer of trajectories [{buf.T}][.][{buf.W}] cannot serve a batch [{T}][{B}][{W}]")
    _expect("slots", dev_slots, torch.int32, (B,))
    _expect_learner_side(T, B, W, learner, values, bootstrap, cfg, out)
    o = _out_struct(out)
    cfg = _cfg_for(cfg, learner)
    _check(load().impact_loss_fwd_bwd_from_buffer(buf.handle, B, _ptr(dev_slots), _ptr(learner), _ptr(values),
                                                  _ptr(bootstrap), ctypes.byref(cfg), ctypes.byref(o),
                                                  _ptr(workspace), workspace.numel(), _stream(stream)),
           "impact_loss_fwd_bwd_from_buffer")
    return out
