"""Python binding of the NNP library: the C ABI's calls under the same names,
a small ``NNPModel`` convenience class, and ``NNPEnergy``, a
torch.autograd.Function whose backward returns -dE/dx from the library's
hand-written adjoint.

Everything here is argument marshalling: device pointers come from torch
CUDA tensors and the stream is torch's current stream; every stage of the
computation runs in the HIP kernels of libnnp.so.
"""
from __future__ import annotations

import ctypes as C

import numpy as np
import torch

from . import _lib as L

__all__ = [
    "NNPError", "nnp_create", "nnp_reserve", "nnp_compute", "nnp_compute_pairs", "nnp_compute_batch", "nnp_compute_noalloc", "nnp_get_status",
    "nnp_read_buffer", "nnp_destroy", "nnp_profile_enable", "nnp_profile_read", "nnp_set_graph", "nnp_autotune", "nnp_set_variant", "nnp_get_variants", "nnp_me_coupling", "nnp_set_links", "nnp_status_string", "nnp_last_error", "nnp_version",
    "make_config", "NNPModel", "NNPEnergy",
]


class NNPError(RuntimeError):
    def __init__(self, status: int, where: str):
        lib = L.load()
        self.status = status
        msg = lib.nnp_last_error().decode() or lib.nnp_status_string(status).decode()
        super().__init__(f"{where}: {lib.nnp_status_string(status).decode()} ({status}): {msg}")


def _check(status: int, where: str) -> None:
    if status != L.NNP_OK:
        raise NNPError(status, where)


# Every call below passes through these three, and 192 atoms take the GPU 42 us:
# plain integers for pointers, the current stream's handle without a Stream
# object (0.4 us instead of 2.8), no copies of arrays that fit as they are.
_current_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream",
                              lambda device: torch.cuda.current_stream(device).cuda_stream)


def _stream(stream) -> int:
    if stream is None:
        return _current_raw_stream(torch.cuda.current_device())
    return int(stream.cuda_stream) if hasattr(stream, "cuda_stream") else int(stream)


def _dptr(t: torch.Tensor | None, dtype: torch.dtype, what: str):
    if t is None:
        return None
    if not t.is_cuda or t.dtype != dtype or not t.is_contiguous():
        raise TypeError(f"{what} must be a contiguous {dtype} CUDA tensor")
    return t.data_ptr()


def _host(a, dtype, what):
    if a is None:
        return None, None
    arr = a if type(a) is np.ndarray and a.dtype == dtype and a.flags.c_contiguous else \
        np.ascontiguousarray(np.asarray(a), dtype=dtype)
    return arr, arr.ctypes.data_as(L._I32P if dtype == np.int32 else L._F32P)


# ----------------------------------------------------------------- raw calls
def nnp_version() -> str:
    return L.load().nnp_version().decode()


def nnp_status_string(s: int) -> str:
    return L.load().nnp_status_string(s).decode()


def nnp_last_error() -> str:
    return L.load().nnp_last_error().decode()


def make_config(cfg: dict, n_members: int = 1):
    """Build the C nnp_config from a hyper-parameter dict.  Returns (struct, keepalive)."""
    keep = []

    def arr(a, dt):
        x = np.ascontiguousarray(np.asarray(a), dtype=dt)
        keep.append(x)
        return x.ctypes.data_as(C.POINTER(C.c_int32 if dt == np.int32 else C.c_float))

    c = L.nnp_config()
    c.n_species = len(cfg["species"])
    c.atomic_numbers_host = arr(cfg["species"], np.int32)
    c.rc_rad, c.rc_ang = float(cfg["rc_rad"]), float(cfg["rc_ang"])
    c.eta_rad, c.eta_ang, c.zeta = float(cfg["eta_rad"]), float(cfg["eta_ang"]), float(cfg["zeta"])
    c.n_rad_shift = len(cfg["rad_shift"])
    c.n_ang_shift = len(cfg["ang_shift"])
    c.n_ang_sect = len(cfg["ang_sect"])
    c.rad_shift_host = arr(cfg["rad_shift"], np.float32)
    c.ang_shift_host = arr(cfg["ang_shift"], np.float32)
    c.ang_sect_host = arr(cfg["ang_sect"], np.float32)
    c.n_layers = len(cfg["widths"])
    c.widths_host = arr(cfg["widths"], np.int32)
    c.celu_alpha = float(cfg["celu_alpha"])
    c.extra_inputs = int(cfg.get("extra_inputs", 0))
    c.mm_cutoff = float(cfg.get("mm_cutoff", 12.0))
    c.ke_coulomb = float(cfg.get("ke_coulomb", 14.3996454784))
    c.n_members = int(n_members)
    return c, keep


def nnp_create(cfg: dict, seed: int = 1, weights=None, precision: str = "fp32", n_members: int = 1) -> C.c_void_p:
    lib = L.load()
    c, keep = make_config(cfg, n_members)
    w, wp = _host(weights, np.float32, "weights") if weights is not None else (None, None)
    h = C.c_void_p()
    prec = {"fp32": L.NNP_FP32, "bf16": L.NNP_BF16}[precision]
    _check(lib.nnp_create(C.byref(c), C.c_uint64(seed), wp, prec, C.byref(h)), "nnp_create")
    del keep, w
    return h


def nnp_reserve(h, max_atoms: int, max_systems: int = 1, max_mm: int = 0, max_rad_nbr: int = 0,
                max_ang_nbr: int = 0) -> None:
    _check(L.load().nnp_reserve(h, max_atoms, max_systems, max_mm, max_rad_nbr, max_ang_nbr), "nnp_reserve")


def nnp_compute(h, pos: torch.Tensor, Z, box, nnp_idx, mm_pos, mm_q, energy: torch.Tensor, forces: torch.Tensor,
                mm_forces=None, accumulate: bool = False, stream=None) -> None:
    n = pos.shape[0]
    Za, Zp = _host(Z, np.int32, "Z")
    Ia, Ip = _host(nnp_idx, np.int32, "nnp_idx")
    Ba, Bp = _host(box, np.float32, "box")
    n_nnp = n if Ia is None else Ia.size
    n_mm = 0 if mm_pos is None else mm_pos.shape[0]
    st = L.load().nnp_compute(h, n, _dptr(pos, torch.float32, "pos"), Zp, Bp, n_nnp, Ip, n_mm,
                              _dptr(mm_pos, torch.float32, "mm_pos"), _dptr(mm_q, torch.float32, "mm_q"),
                              _dptr(energy, torch.float64, "energy"), _dptr(forces, torch.float64, "forces"),
                              _dptr(mm_forces, torch.float64, "mm_forces"), 1 if accumulate else 0,
                              _stream(stream))
    _check(st, "nnp_compute")


KE_COULOMB = 14.3996454784   # eV * A / e^2


def nnp_me_coupling(ml_pos: torch.Tensor, ml_param: torch.Tensor, mm_pos: torch.Tensor, mm_param: torch.Tensor,
                    box=None, cutoff: float = 12.0, ke: float = KE_COULOMB, accumulate: bool = False, out=None,
                    stream=None):
    """Mechanical-embedding ML-MM coupling (eq. 3): Coulomb + Lennard-Jones over ML x MM pairs.

    Params are [n, 3] FP32 CUDA tensors of (q, sigma, eps).  Returns (E [1], F_ml, F_mm) FP64
    tensors (new ones unless `out` supplies them; with accumulate=True they are added to)."""
    n_ml, n_mm = ml_pos.shape[0], mm_pos.shape[0]
    dev = ml_pos.device if n_ml else mm_pos.device
    if out is None:
        E = torch.zeros(1, dtype=torch.float64, device=dev)
        Fml = torch.zeros((n_ml, 3), dtype=torch.float64, device=dev)
        Fmm = torch.zeros((n_mm, 3), dtype=torch.float64, device=dev)
    else:
        E, Fml, Fmm = out
    Ba, Bp = _host(box, np.float32, "box")
    st = L.load().nnp_me_coupling(n_ml, _dptr(ml_pos, torch.float32, "ml_pos"),
                                  _dptr(ml_param, torch.float32, "ml_param"), n_mm,
                                  _dptr(mm_pos, torch.float32, "mm_pos"), _dptr(mm_param, torch.float32, "mm_param"),
                                  Bp, float(cutoff), float(ke), _dptr(E, torch.float64, "energy"),
                                  _dptr(Fml, torch.float64, "ml_forces"), _dptr(Fmm, torch.float64, "mm_forces"),
                                  1 if accumulate else 0, _stream(stream))
    _check(st, "nnp_me_coupling")
    return E, Fml, Fmm


def nnp_compute_pairs(h, pos: torch.Tensor, Z, box, nnp_idx, pairs: torch.Tensor, mm_pos, mm_q,
                      energy: torch.Tensor, forces: torch.Tensor, mm_forces=None, accumulate: bool = False,
                      stream=None) -> None:
    """nnp_compute with the neighbour lists taken from a caller's [n_pairs, 2] int32 CUDA pair list."""
    n = pos.shape[0]
    Za, Zp = _host(Z, np.int32, "Z")
    Ia, Ip = _host(nnp_idx, np.int32, "nnp_idx")
    Ba, Bp = _host(box, np.float32, "box")
    n_nnp = n if Ia is None else Ia.size
    n_mm = 0 if mm_pos is None else mm_pos.shape[0]
    st = L.load().nnp_compute_pairs(h, n, _dptr(pos, torch.float32, "pos"), Zp, Bp, n_nnp, Ip, pairs.shape[0],
                                    _dptr(pairs, torch.int32, "pairs"), n_mm,
                                    _dptr(mm_pos, torch.float32, "mm_pos"), _dptr(mm_q, torch.float32, "mm_q"),
                                    _dptr(energy, torch.float64, "energy"), _dptr(forces, torch.float64, "forces"),
                                    _dptr(mm_forces, torch.float64, "mm_forces"), 1 if accumulate else 0,
                                    _stream(stream))
    _check(st, "nnp_compute_pairs")


def nnp_compute_batch(h, offsets, pos: torch.Tensor, Z, energies: torch.Tensor, forces: torch.Tensor,
                      boxes=None, stream=None) -> None:
    """Packed systems; boxes: None (all open) or [n_sys, 3] lengths, a zero row for an open system."""
    Oa, Op = _host(offsets, np.int32, "offsets")
    Za, Zp = _host(Z, np.int32, "Z")
    Ba, Bp = _host(None if boxes is None else np.asarray(boxes, np.float32).reshape(-1), np.float32, "boxes")
    st = L.load().nnp_compute_batch(h, Oa.size - 1, Op, _dptr(pos, torch.float32, "pos"), Zp, Bp,
                                    _dptr(energies, torch.float64, "energies"),
                                    _dptr(forces, torch.float64, "forces"), _stream(stream))
    _check(st, "nnp_compute_batch")


def nnp_compute_noalloc(h, pos: torch.Tensor, Z, box, energy: torch.Tensor, forces: torch.Tensor,
                        stream=None) -> None:
    """nnp_compute for an all-NNP system on the library's static workspace (allocates nothing)."""
    n = pos.shape[0]
    Za, Zp = _host(Z, np.int32, "Z")
    Ba, Bp = _host(box, np.float32, "box")
    st = L.load().nnp_compute_noalloc(h, n, _dptr(pos, torch.float32, "pos"), Zp, Bp,
                                      _dptr(energy, torch.float64, "energy"), _dptr(forces, torch.float64, "forces"),
                                      _stream(stream))
    _check(st, "nnp_compute_noalloc")


def nnp_get_status(h, stream=None) -> int:
    return L.load().nnp_get_status(h, _stream(stream))


def nnp_read_buffer(h, which: int, stream=None) -> np.ndarray:
    lib = L.load()
    elems = C.c_int64()
    stride = C.c_int32()
    _check(lib.nnp_read_buffer(h, which, None, 0, C.byref(elems), C.byref(stride), _stream(stream)),
           "nnp_read_buffer")
    dt = (np.float32 if which in (L.NNP_BUF_DESCRIPTOR, L.NNP_BUF_ATOM_ENERGY, L.NNP_BUF_DEDX, L.NNP_BUF_CHARGE)
          else np.int32)
    out = np.empty(elems.value, dtype=dt)
    _check(lib.nnp_read_buffer(h, which, out.ctypes.data_as(C.c_void_p), out.nbytes, C.byref(elems),
                               C.byref(stride), _stream(stream)), "nnp_read_buffer")
    if stride.value > 1:
        out = out.reshape(-1, stride.value)
    return out


def nnp_autotune(h, reps: int = 5, stream=None) -> dict:
    """Time every kernel variant on the last call's workspace and keep the fastest."""
    chosen = (C.c_int32 * 4)()
    _check(L.load().nnp_autotune(h, int(reps), chosen, _stream(stream)), "nnp_autotune")
    return {k: chosen[v] for k, v in TUNE_STAGES.items()}


TUNE_STAGES = {"neighbours": 0, "descriptor": 1, "network": 2, "adjoint": 3}


def nnp_get_variants(h) -> dict:
    """Kernel variants a call of the previous call's size and geometry runs."""
    chosen = (C.c_int32 * 4)()
    _check(L.load().nnp_get_variants(h, chosen), "nnp_get_variants")
    return {k: chosen[v] for k, v in TUNE_STAGES.items()}


def nnp_set_variant(h, stage, variant: int) -> None:
    """Pin a stage's kernel variant (-1: tuned choice / default); stage by name or number."""
    st = TUNE_STAGES[stage] if isinstance(stage, str) else int(stage)
    _check(L.load().nnp_set_variant(h, st, int(variant)), "nnp_set_variant")


def nnp_set_links(h, ml_idx, mm_idx, distance: float = 1.0, link_Z: int = 1) -> None:
    """Link atoms on the bonds ml_idx[l] (inside the index group) -> mm_idx[l] (outside), eq. 4."""
    ml, mlp = _host(ml_idx, np.int32, "ml_idx")
    mm, mmp = _host(mm_idx, np.int32, "mm_idx")
    n = 0 if ml is None else ml.size
    _check(L.load().nnp_set_links(h, n, mlp, mmp, float(distance), int(link_Z)), "nnp_set_links")


def nnp_set_graph(h, enable: bool) -> None:
    _check(L.load().nnp_set_graph(h, 1 if enable else 0), "nnp_set_graph")


def nnp_profile_enable(h, max_calls: int) -> None:
    _check(L.load().nnp_profile_enable(h, int(max_calls)), "nnp_profile_enable")


def nnp_profile_read(h, stream=None) -> tuple[dict, int]:
    """Summed per-stage event times (ms) over the recorded calls, and the call count."""
    ms = (C.c_double * L.NNP_STAGE_COUNT)()
    calls = C.c_int64()
    _check(L.load().nnp_profile_read(h, ms, C.byref(calls), _stream(stream)), "nnp_profile_read")
    return {name: ms[k] for k, name in enumerate(L.STAGES)}, calls.value


def nnp_destroy(h) -> None:
    L.load().nnp_destroy(h)


# ------------------------------------------------------------ convenience
class NNPModel:
    """Owns one library model on the current device."""

    def __init__(self, cfg: dict, seed: int = 1, weights=None, precision: str = "fp32", n_members: int = 1):
        self.cfg = cfg
        self.precision = precision
        self.h = nnp_create(cfg, seed, weights, precision, n_members)
        self.capacity = None

    def reserve(self, max_atoms: int, max_systems: int = 1, max_mm: int = 0, max_rad_nbr: int = 0,
                max_ang_nbr: int = 0) -> None:
        nnp_reserve(self.h, max_atoms, max_systems, max_mm, max_rad_nbr, max_ang_nbr)
        self.capacity = (max_atoms, max_systems, max_mm, max_rad_nbr, max_ang_nbr)

    def _ensure(self, n_atoms: int, n_sys: int = 1, n_mm: int = 0) -> None:
        c = self.capacity
        if c is None or n_atoms > c[0] or n_sys > c[1] or n_mm > c[2]:
            base = c if c is not None else (0, 1, 0, 0, 0)
            self.reserve(max(n_atoms, base[0]), max(n_sys, base[1]), max(n_mm, base[2]), base[3], base[4])

    def compute(self, pos: torch.Tensor, Z=None, box=None, nnp_idx=None, mm_pos=None, mm_q=None,
                accumulate_into=None, out=None, stream=None):
        """Energy [1] (float64) and forces [n, 3] (float64) on pos.device; MM forces if MM charges are given.

        Z=None reuses the topology of the previous call.  ``out=(E, F, F_mm)`` writes into
        preallocated tensors; ``accumulate_into=(E, F, F_mm)`` adds to them instead.
        """
        n = pos.shape[0]
        self._ensure(n, 1, 0 if mm_pos is None else mm_pos.shape[0])
        dev = pos.device
        if accumulate_into is not None:
            E, F, Fmm = accumulate_into
        elif out is not None:
            E, F, Fmm = out
        else:
            E = torch.empty(1, dtype=torch.float64, device=dev)
            F = torch.empty((n, 3), dtype=torch.float64, device=dev)
            Fmm = None if mm_pos is None else torch.empty((mm_pos.shape[0], 3), dtype=torch.float64, device=dev)
        nnp_compute(self.h, pos, Z, box, nnp_idx, mm_pos, mm_q, E, F, Fmm,
                    accumulate=accumulate_into is not None, stream=stream)
        return E, F, Fmm

    def compute_pairs(self, pos: torch.Tensor, pairs: torch.Tensor, Z=None, box=None, nnp_idx=None, mm_pos=None,
                      mm_q=None, out=None, stream=None):
        """As compute, with the neighbour lists built from a [n_pairs, 2] int32 CUDA half pair list."""
        n = pos.shape[0]
        self._ensure(n, 1, 0 if mm_pos is None else mm_pos.shape[0])
        dev = pos.device
        if out is not None:
            E, F, Fmm = out
        else:
            E = torch.empty(1, dtype=torch.float64, device=dev)
            F = torch.empty((n, 3), dtype=torch.float64, device=dev)
            Fmm = None if mm_pos is None else torch.empty((mm_pos.shape[0], 3), dtype=torch.float64, device=dev)
        nnp_compute_pairs(self.h, pos, Z, box, nnp_idx, pairs, mm_pos, mm_q, E, F, Fmm, stream=stream)
        return E, F, Fmm

    def compute_batch(self, pos: torch.Tensor, Z, offsets, boxes=None, out=None, stream=None):
        """Per-system energies [n_sys] and forces [n, 3] (float64) of packed systems (boxes: None = all
        open, or [n_sys, 3] box lengths with zero rows for open systems)."""
        offsets = np.asarray(offsets, dtype=np.int32)
        self._ensure(pos.shape[0], offsets.size - 1)
        if out is not None:
            E, F = out
        else:
            E = torch.empty(offsets.size - 1, dtype=torch.float64, device=pos.device)
            F = torch.empty((pos.shape[0], 3), dtype=torch.float64, device=pos.device)
        nnp_compute_batch(self.h, offsets, pos, Z, E, F, boxes=boxes, stream=stream)
        return E, F

    def set_graph(self, enable: bool) -> None:
        nnp_set_graph(self.h, enable)

    def set_links(self, ml_idx, mm_idx, distance: float = 1.0, link_Z: int = 1) -> None:
        nnp_set_links(self.h, ml_idx, mm_idx, distance, link_Z)

    def autotune(self, reps: int = 5) -> dict:
        return nnp_autotune(self.h, reps)

    def set_variant(self, stage, variant: int) -> None:
        nnp_set_variant(self.h, stage, variant)

    def variants(self) -> dict:
        return nnp_get_variants(self.h)

    def status(self, stream=None) -> int:
        return nnp_get_status(self.h, stream)

    def read(self, which: int) -> np.ndarray:
        return nnp_read_buffer(self.h, which)

    def _autograd_outputs(self, pos: torch.Tensor):
        """Output buffers the autograd path reuses call after call (same size, same device)."""
        key = (pos.shape[0], pos.device)
        buf = getattr(self, "_ag_buf", None)
        if buf is None or buf[0] != key:
            E = torch.empty(1, dtype=torch.float64, device=pos.device)
            F = torch.empty((pos.shape[0], 3), dtype=torch.float64, device=pos.device)
            self._ag_buf = buf = (key, (E, F, None))
        return buf[1]

    def energy(self, pos: torch.Tensor, Z=None, box=None, nnp_idx=None):
        """Differentiable E_ML(pos): backward gives -forces via the library's adjoint."""
        return NNPEnergy.apply(pos, self, Z, box, nnp_idx)

    def close(self) -> None:
        if self.h:
            nnp_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class NNPEnergy(torch.autograd.Function):
    """E = NNPEnergy.apply(pos, model, Z, box, nnp_idx); dE/dpos = -F from the same call.

    The library writes into the model's persistent output buffers (so repeated
    calls replay one captured graph); the returned energy and the saved gradient
    are copies of them."""

    @staticmethod
    def forward(ctx, pos, model, Z, box, nnp_idx):
        p = pos.detach()
        if p.dtype != torch.float32:
            p = p.float()
        E, F, _ = model.compute(p.contiguous(), Z, box, nnp_idx, out=model._autograd_outputs(p))
        ctx.save_for_backward(F.neg())
        ctx.in_dtype = pos.dtype
        return E[0].clone()

    @staticmethod
    def backward(ctx, gE):
        (G,) = ctx.saved_tensors
        return (gE.to(torch.float64) * G).to(ctx.in_dtype), None, None, None, None
