"""ctypes binding of libfqpd.so (the C ABI in include/fqpd.h).

Argument marshalling only: every entry point takes torch tensors that already live
on the GPU, passes their device pointers and the current HIP stream, and raises
FqError when the library returns a non-OK status.  All arithmetic runs in the HIP
kernels; there is no CPU fallback.  The library must have been built in-tree
(paper_2509_05464_amd.build.build()); loading fails loudly otherwise.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence, Tuple

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, 'libfqpd.so')

FQ_MAX_ANGLES = 32
FQ_MAX_NT = 512
FQ_SSM_MAX_MODES = 64
CUTOFF_KNEE, CUTOFF_SSM = -1, -2
DISP_POWER, DISP_IQ, DISP_UNIT = 0, 1, 2
MIP_XY, MIP_XZ, MIP_YZ = 0, 1, 2
LCF_N_PARAM = 19170
FQ_OK, FQ_E_INVALID, FQ_E_WORKSPACE, FQ_E_HIP, FQ_E_NUMERIC = range(5)
INTERP_LINEAR, INTERP_HERMITE = 0, 1
GRAM_FP32, GRAM_SPLIT_BF16, GRAM_BF16, GRAM_SPLIT4_BF16 = 0, 1, 2, 3


class FqError(RuntimeError):
    def __init__(self, fn: str, status: int, msg: str):
        super().__init__(f'{fn} failed with status {status}: {msg}')
        self.status = status


class Probe(ctypes.Structure):
    _fields_ = [('nx_el', ctypes.c_int32), ('ny_el', ctypes.c_int32),
                ('pitch_x', ctypes.c_double), ('pitch_y', ctypes.c_double),
                ('fc_hz', ctypes.c_double), ('fs_hz', ctypes.c_double), ('c_mps', ctypes.c_double)]


class Tx(ctypes.Structure):
    _fields_ = [('n_angles', ctypes.c_int32), ('tilt_rad', (ctypes.c_double * 2) * FQ_MAX_ANGLES)]


class Grid(ctypes.Structure):
    _fields_ = [('nx', ctypes.c_int32), ('ny', ctypes.c_int32), ('nz', ctypes.c_int32),
                ('x0', ctypes.c_double), ('y0', ctypes.c_double), ('z0', ctypes.c_double),
                ('dx', ctypes.c_double), ('dy', ctypes.c_double), ('dz', ctypes.c_double)]


class Pulse(ctypes.Structure):
    _fields_ = [('n_cycles', ctypes.c_double), ('trunc_sigmas', ctypes.c_double), ('r_ref_m', ctypes.c_double)]


class FdParams(ctypes.Structure):
    _fields_ = [('elem_width_x', ctypes.c_double), ('elem_width_y', ctypes.c_double),
                ('n_sub_x', ctypes.c_int32), ('n_sub_y', ctypes.c_int32),
                ('atten_db_cm_mhz', ctypes.c_double), ('spectral_floor', ctypes.c_double)]


def make_fd_params(elem_width=(0.0, 0.0), n_sub=(1, 1), atten_db_cm_mhz=0.0, spectral_floor=1e-7) -> FdParams:
    return FdParams(elem_width[0], elem_width[1], n_sub[0], n_sub[1], atten_db_cm_mhz, spectral_floor)


WS_DAS, WS_DAS_MIN, WS_GRAM, WS_SVD, WS_SSM, WS_FD, WS_DISPLAY, WS_FALLBACK, WS_LCF_ACT = range(9)


class WsQuery(ctypes.Structure):
    _fields_ = [('probe', ctypes.POINTER(Probe)), ('tx', ctypes.POINTER(Tx)), ('pulse', ctypes.POINTER(Pulse)),
                ('fd', ctypes.POINTER(FdParams)), ('n', ctypes.c_int64), ('n_t', ctypes.c_int32),
                ('n_samples', ctypes.c_int32), ('gram_mode', ctypes.c_int32)]


def make_probe(nx_el, ny_el, pitch_x, pitch_y, fc, fs, c) -> Probe:
    return Probe(nx_el, ny_el, pitch_x, pitch_y, fc, fs, c)


def make_tx(tilts_rad: Sequence[Tuple[float, float]]) -> Tx:
    t = Tx()
    if not 1 <= len(tilts_rad) <= FQ_MAX_ANGLES:
        raise ValueError('1..32 transmits')
    t.n_angles = len(tilts_rad)
    for i, (a, b) in enumerate(tilts_rad):
        t.tilt_rad[i][0] = a
        t.tilt_rad[i][1] = b
    return t


def make_grid(nx, ny, nz, x0, y0, z0, dx, dy, dz) -> Grid:
    return Grid(nx, ny, nz, x0, y0, z0, dx, dy, dz)


def make_pulse(n_cycles=2.0, trunc_sigmas=5.0, r_ref=1e-3) -> Pulse:
    return Pulse(n_cycles, trunc_sigmas, r_ref)


_lib: Optional[ctypes.CDLL] = None

_P = ctypes.POINTER
_vp, _i32, _i64, _f32, _sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t

_SIGS = {
    'rf_synth': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Pulse), _i32, _i64, _vp, _i32, _vp, _i32, _i32, _vp, _vp]),
    'fd_workspace_size': (_sz, [_P(Probe), _P(Tx), _P(Pulse), _P(FdParams), _i32, _i64]),
    'fd_synth': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Pulse), _P(FdParams), _i32, _i64, _vp, _i32, _vp, _vp, _i32, _i32,
                                _vp, _sz, _vp, _vp]),
    'das_workspace_size': (_sz, [_P(Probe), _P(Tx), _i32, _i32, _i32]),
    'das_beamform': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Grid), _i32, _i32, _vp, _i32, _vp, _sz, _vp, _vp]),
    'das_demodulate': (ctypes.c_int, [_P(Probe), _P(Tx), _i32, _i32, _vp, _vp, _sz, _vp]),
    'das_delay_sum': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Grid), _i32, _i32, _i32, _vp, _sz, _vp, _vp]),
    'das_window_rows': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Grid)]),
    'das_launch_shape': (ctypes.c_int, [_P(Probe), _P(Tx), _P(Grid), _i32, _i32, _i32, _P(_i64)]),
    'gram_workspace_size': (_sz, [_i64, _i32, _i32]),
    'casorati_gram': (ctypes.c_int, [_vp, _i64, _i32, _i32, _vp, _sz, _vp, _vp]),
    'casorati_gram_noalloc': (ctypes.c_int, [_vp, _i64, _i32, _i32, _vp, _vp]),
    'svd_workspace_size': (_sz, [_i64, _i32]),
    'svd_clutter_filter': (ctypes.c_int, [_vp, _i64, _i32, _vp, _i32, _vp, _sz, _vp, _vp, _vp, _vp, _vp, _vp]),
    'svd_filter_apply': (ctypes.c_int, [_vp, _i64, _i32, _vp, _sz, _vp, _vp, _vp, _vp]),
    'hermitian_eig': (ctypes.c_int, [_vp, _i32, _vp, _sz, _vp, _vp, _vp, _vp]),
    'power_doppler': (ctypes.c_int, [_vp, _i64, _i32, _vp, _vp]),
    'ssm_workspace_size': (_sz, [_i64, _i32]),
    'display_workspace_size': (_sz, [_i64]),
    'display_db': (ctypes.c_int, [_vp, _i64, _i32, _f32, _vp, _sz, _vp, _vp, _vp]),
    'mip': (ctypes.c_int, [_vp, _i32, _i32, _i32, _i32, _vp, _vp]),
    'image_quality': (ctypes.c_int, [_vp, _vp, _i32, _i32, ctypes.c_double, _vp, _vp]),
    'spatial_similarity': (ctypes.c_int, [_vp, _i64, _i32, _vp, _i32, _vp, _sz, _vp, _vp, _vp]),
    'lcf_act_size': (_sz, [_i64, _i32]),
    'lcf_forward': (ctypes.c_int, [_vp, _vp, _vp, _i64, _i32, _f32, _vp, _vp, _vp, _vp]),
    'lcf_backward': (ctypes.c_int, [_vp, _vp, _vp, _vp, _i64, _i32, _f32, _vp, _vp, _vp, _vp]),
    'lcf_adam_step': (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, _i32, _f32, _f32, _f32, _f32, _i32, _vp]),
    'lcf_gather': (ctypes.c_int, [_vp, _i64, _i32, _i64, _vp, _i64, _vp, _vp]),
    'fallback_workspace_size': (_sz, [_i64]),
    'lcf_fallback': (ctypes.c_int, [_vp, _vp, _i64, _f32, _vp, _sz, _vp, _vp, _vp, _vp]),
    'fq_workspace_size': (_sz, [_i32, _vp]),
    'roof_probe': (ctypes.c_int, [_i32, _i32, _i32, _vp, _vp]),
    'fq_version': (ctypes.c_int, []),
    'fq_last_error': (ctypes.c_char_p, []),
}


def lib() -> ctypes.CDLL:
    """Load the in-tree libfqpd.so; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f'{LIB_PATH} is missing: build it with paper_2509_05464_amd.build.build()')
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _ptr(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError('expected a GPU tensor')
    if not t.is_contiguous():
        raise ValueError('expected a contiguous tensor')
    return ctypes.c_void_p(t.data_ptr())


def _check(name: str, st: int):
    if st != FQ_OK:
        raise FqError(name, st, lib().fq_last_error().decode())


def _f32view(t: torch.Tensor) -> torch.Tensor:
    return torch.view_as_real(t) if t.is_complex() else t


# ----------------------------------------------------------------------------- stages
def rf_synth(probe: Probe, tx: Tx, pulse: Pulse, pos: torch.Tensor, amp: torch.Tensor, rf: torch.Tensor,
             pos_static: bool = False, accumulate: bool = False) -> None:
    """rf float32 [F][A][E][T]; pos float32 [F or 1][S][3]; amp float32 [S]."""
    F, A, E, T = rf.shape
    S = amp.numel()
    st = lib().rf_synth(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(pulse), F, S, _ptr(pos),
                        int(pos_static), _ptr(amp), T, int(accumulate), _ptr(rf), _stream())
    _check('rf_synth', st)


def fd_workspace_size(probe: Probe, tx: Tx, pulse: Pulse, fdp: FdParams, n_samples: int,
                      scatterers_per_block: int) -> int:
    return lib().fd_workspace_size(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(pulse), ctypes.byref(fdp),
                                   n_samples, scatterers_per_block)


def fd_synth(probe: Probe, tx: Tx, pulse: Pulse, fdp: FdParams, pos: torch.Tensor, amp: torch.Tensor,
             rf: torch.Tensor, ws: torch.Tensor, pos_static: bool = False, accumulate: bool = False,
             apod: Optional[torch.Tensor] = None) -> None:
    """pos float32 [F or 1][S][3], amp [S] -> rf float32 [F][A][E][T] (frequency-domain model)."""
    F, A, E, T = rf.shape
    n_scat = amp.numel()
    st = lib().fd_synth(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(pulse), ctypes.byref(fdp), F, n_scat,
                        _ptr(pos) if n_scat else None, int(pos_static), _ptr(amp) if n_scat else None, _ptr(apod), T,
                        int(accumulate), _ptr(ws), ws.numel() * ws.element_size(), _ptr(rf), _stream())
    _check('fd_synth', st)


def das_workspace_size(probe: Probe, tx: Tx, n_frames: int, n_samples: int, minimum: bool = False) -> int:
    return lib().das_workspace_size(ctypes.byref(probe), ctypes.byref(tx), n_frames, n_samples, int(minimum))


def das_window_rows(probe: Probe, tx: Tx, grid: Grid) -> int:
    """Delay rows staged on chip per (transmit, element) for one voxel tile (host query)."""
    w = lib().das_window_rows(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(grid))
    if w < 0:
        _check("das_window_rows", FQ_E_INVALID)
    return int(w)


def das_launch_shape(probe: Probe, tx: Tx, grid: Grid, n_frames: int, n_samples: int,
                     interp: int = INTERP_LINEAR) -> Tuple[int, ...]:
    """(frames of a block, transmits of a pass, element groups, wide windows, voxel tiles) of a call (host query)."""
    shape = (_i64 * 5)()
    _check('das_launch_shape', lib().das_launch_shape(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(grid), n_frames,
                                                      n_samples, interp, shape))
    return tuple(shape)


def das_beamform(probe: Probe, tx: Tx, grid: Grid, rf: torch.Tensor, iq: torch.Tensor, ws: torch.Tensor,
                 interp: int = INTERP_LINEAR) -> None:
    """rf float32 [F][A][E][T] -> iq complex64 [F][Nv]."""
    F, A, E, T = rf.shape
    st = lib().das_beamform(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(grid), F, T, _ptr(rf), interp,
                            _ptr(ws), ws.numel() * ws.element_size(), _ptr(_f32view(iq)), _stream())
    _check('das_beamform', st)


def das_demodulate(probe: Probe, tx: Tx, rf: torch.Tensor, ws: torch.Tensor) -> None:
    F, A, E, T = rf.shape
    st = lib().das_demodulate(ctypes.byref(probe), ctypes.byref(tx), F, T, _ptr(rf), _ptr(ws),
                              ws.numel() * ws.element_size(), _stream())
    _check('das_demodulate', st)


def das_delay_sum(probe: Probe, tx: Tx, grid: Grid, n_samples: int, ws: torch.Tensor, iq: torch.Tensor,
                  interp: int = INTERP_LINEAR) -> None:
    F = iq.shape[0]
    st = lib().das_delay_sum(ctypes.byref(probe), ctypes.byref(tx), ctypes.byref(grid), F, n_samples, interp,
                             _ptr(ws), ws.numel() * ws.element_size(), _ptr(_f32view(iq)), _stream())
    _check('das_delay_sum', st)


def fq_workspace_size(which: int, probe: Optional[Probe] = None, tx: Optional[Tx] = None,
                      pulse: Optional[Pulse] = None, fdp: Optional[FdParams] = None, n: int = 0, n_t: int = 0,
                      n_samples: int = 0, gram_mode: int = GRAM_FP32) -> int:
    """The one workspace query of the library (WS_* selects the entry point)."""
    q = WsQuery()
    q.probe = ctypes.pointer(probe) if probe is not None else None
    q.tx = ctypes.pointer(tx) if tx is not None else None
    q.pulse = ctypes.pointer(pulse) if pulse is not None else None
    q.fd = ctypes.pointer(fdp) if fdp is not None else None
    q.n, q.n_t, q.n_samples, q.gram_mode = n, n_t, n_samples, gram_mode
    return lib().fq_workspace_size(which, ctypes.byref(q))


def gram_workspace_size(n_vox: int, n_t: int, mode: int = GRAM_FP32) -> int:
    return lib().gram_workspace_size(n_vox, n_t, mode)


def casorati_gram(iq: torch.Tensor, gram: torch.Tensor, ws: torch.Tensor, mode: int = GRAM_FP32) -> None:
    """iq complex64 [Nt][Nv] -> gram complex128 [Nt][Nt]."""
    nt, nv = iq.shape
    st = lib().casorati_gram(_ptr(_f32view(iq)), nv, nt, mode, _ptr(ws), ws.numel() * ws.element_size(),
                             _ptr(_f32view(gram)), _stream())
    _check('casorati_gram', st)


PROBE_LDS_READ, PROBE_FP32_FMA = 0, 1


def roof_probe(which: int, out: torch.Tensor, iters: int) -> None:
    """Launch an on-chip ceiling probe over out.numel() / 256 workgroups (measurement helper)."""
    n_blocks = out.numel() // 256
    st = lib().roof_probe(which, n_blocks, iters, _ptr(out), _stream())
    _check('roof_probe', st)


def casorati_gram_noalloc(iq: torch.Tensor, gram: torch.Tensor, mode: int = GRAM_FP32) -> None:
    """casorati_gram without a workspace (the library's static scratch array)."""
    nt, nv = iq.shape
    st = lib().casorati_gram_noalloc(_ptr(_f32view(iq)), nv, nt, mode, _ptr(_f32view(gram)), _stream())
    _check('casorati_gram_noalloc', st)


def svd_workspace_size(n_vox: int, n_t: int) -> int:
    return lib().svd_workspace_size(n_vox, n_t)


def svd_clutter_filter(iq: torch.Tensor, gram: torch.Tensor, ws: torch.Tensor, sigma: torch.Tensor,
                       k_used: torch.Tensor, cutoff: int = -1, iq_filt: Optional[torch.Tensor] = None,
                       pd: Optional[torch.Tensor] = None, status: Optional[torch.Tensor] = None) -> None:
    nt, nv = iq.shape
    st = lib().svd_clutter_filter(_ptr(_f32view(iq)), nv, nt, _ptr(_f32view(gram)), cutoff, _ptr(ws),
                                  ws.numel() * ws.element_size(),
                                  _ptr(_f32view(iq_filt)) if iq_filt is not None else None,
                                  _ptr(pd), _ptr(sigma), _ptr(k_used), _ptr(status), _stream())
    _check('svd_clutter_filter', st)


def svd_filter_apply(iq: torch.Tensor, ws: torch.Tensor, k_used: torch.Tensor, iq_filt: Optional[torch.Tensor] = None,
                     pd: Optional[torch.Tensor] = None) -> None:
    """Projection and power Doppler from the V_K and K a svd_clutter_filter call left in ws."""
    nt, nv = iq.shape
    st = lib().svd_filter_apply(_ptr(_f32view(iq)), nv, nt, _ptr(ws), ws.numel() * ws.element_size(), _ptr(k_used),
                                _ptr(_f32view(iq_filt)) if iq_filt is not None else None, _ptr(pd), _stream())
    _check('svd_filter_apply', st)


def hermitian_eig(gram: torch.Tensor, ws: torch.Tensor, lam: torch.Tensor, vecs: Optional[torch.Tensor] = None,
                  status: Optional[torch.Tensor] = None) -> None:
    nt = gram.shape[0]
    st = lib().hermitian_eig(_ptr(_f32view(gram)), nt, _ptr(ws), ws.numel() * ws.element_size(), _ptr(lam),
                             _ptr(_f32view(vecs)) if vecs is not None else None, _ptr(status), _stream())
    _check('hermitian_eig', st)


def power_doppler(iq: torch.Tensor, pd: torch.Tensor) -> None:
    nt, nv = iq.shape
    st = lib().power_doppler(_ptr(_f32view(iq)), nv, nt, _ptr(pd), _stream())
    _check('power_doppler', st)


def ssm_workspace_size(n_vox: int, n_t: int) -> int:
    return lib().ssm_workspace_size(n_vox, n_t)


def spatial_similarity(iq: torch.Tensor, vecs: torch.Tensor, n_modes: int, ws: torch.Tensor, ssm: torch.Tensor,
                       k_tissue: Optional[torch.Tensor] = None) -> None:
    """iq complex64 [Nt][Nv], vecs complex128 [Nt][Nt] -> ssm float64 [M][M], k_tissue int32 [1]."""
    nt, nv = iq.shape
    st = lib().spatial_similarity(_ptr(_f32view(iq)), nv, nt, _ptr(_f32view(vecs)), n_modes, _ptr(ws),
                                  ws.numel() * ws.element_size(), _ptr(ssm), _ptr(k_tissue), _stream())
    _check('spatial_similarity', st)


def display_workspace_size(n: int) -> int:
    return lib().display_workspace_size(n)


def display_db(x: torch.Tensor, dr_db: float, ws: torch.Tensor, out: torch.Tensor,
               peak: Optional[torch.Tensor] = None, unit: bool = False) -> None:
    """x float32 power values or complex64 IQ (any shape, contiguous) -> out float32 dB, same
    shape (unit=True: grey levels 1 + dB / dr_db in [0, 1])."""
    kind = (DISP_IQ if x.is_complex() else DISP_POWER) | (DISP_UNIT if unit else 0)
    st = lib().display_db(_ptr(_f32view(x)), x.numel(), kind, dr_db, _ptr(ws), ws.numel() * ws.element_size(),
                          _ptr(out), _ptr(peak), _stream())
    _check('display_db', st)


def mip(vol: torch.Tensor, plane: int, out: torch.Tensor) -> None:
    """vol float32 [nz][ny][nx] -> out: MIP_XY [ny][nx], MIP_XZ [nz][nx], MIP_YZ [nz][ny]."""
    nz, ny, nx = vol.shape
    st = lib().mip(_ptr(vol), nx, ny, nz, plane, _ptr(out), _stream())
    _check('mip', st)


def image_quality(img: torch.Tensor, ref: torch.Tensor, out: torch.Tensor, data_range: float = 1.0) -> None:
    """img, ref float32 [ny][nx] -> out float64 [3] = (MSE, PSNR, SSIM)."""
    ny, nx = img.shape
    if ref.shape != img.shape:
        raise ValueError('img and ref differ in shape')
    st = lib().image_quality(_ptr(img), _ptr(ref), nx, ny, data_range, _ptr(out), _stream())
    _check('image_quality', st)


# ----------------------------------------------------------------------------- learned filter
def lcf_act_size(n_series: int, n_t: int) -> int:
    return lib().lcf_act_size(n_series, n_t)


def lcf_forward(w: torch.Tensor, w_bf16: torch.Tensor, x: torch.Tensor, eps: float = 1e-30,
                act: Optional[torch.Tensor] = None, y: Optional[torch.Tensor] = None,
                pd: Optional[torch.Tensor] = None) -> None:
    nt, n = x.shape
    st = lib().lcf_forward(_ptr(w), _ptr(w_bf16), _ptr(_f32view(x)), n, nt, eps, _ptr(act),
                           _ptr(_f32view(y)) if y is not None else None, _ptr(pd), _stream())
    _check('lcf_forward', st)


def lcf_backward(w: torch.Tensor, w_bf16: torch.Tensor, x: torch.Tensor, target: torch.Tensor, act: torch.Tensor,
                 grad: torch.Tensor, loss: torch.Tensor, eps: float = 1e-30) -> None:
    nt, n = x.shape
    st = lib().lcf_backward(_ptr(w), _ptr(w_bf16), _ptr(_f32view(x)), _ptr(_f32view(target)), n, nt, eps,
                            _ptr(act), _ptr(grad), _ptr(loss), _stream())
    _check('lcf_backward', st)


def lcf_adam_step(w: torch.Tensor, w_bf16: torch.Tensor, m: torch.Tensor, v: torch.Tensor, grad: torch.Tensor,
                  step: int, lr: float = 1e-3, beta1: float = 0.9, beta2: float = 0.999, eps: float = 1e-8) -> None:
    st = lib().lcf_adam_step(_ptr(w), _ptr(w_bf16), _ptr(m), _ptr(v), _ptr(grad), w.numel(), lr, beta1, beta2, eps,
                             step, _stream())
    _check('lcf_adam_step', st)


def lcf_gather(src: torch.Tensor, idx: torch.Tensor, dst: torch.Tensor) -> None:
    """src complex64 [n_vol][Nt][Nv], idx int64 [B] -> dst complex64 [Nt][B]."""
    n_vol, nt, nv = src.shape
    st = lib().lcf_gather(_ptr(_f32view(src)), nv, nt, n_vol, _ptr(idx), idx.numel(), _ptr(_f32view(dst)),
                          _stream())
    _check('lcf_gather', st)


def fallback_workspace_size(n: int) -> int:
    return lib().fallback_workspace_size(n)


def lcf_fallback(pd_l: torch.Tensor, pd_s: torch.Tensor, out: torch.Tensor, flag: torch.Tensor, d_db: torch.Tensor,
                 ws: torch.Tensor, tau_db: float = -10.0) -> None:
    st = lib().lcf_fallback(_ptr(pd_l), _ptr(pd_s), pd_l.numel(), tau_db, _ptr(ws), ws.numel() * ws.element_size(),
                            _ptr(out), _ptr(flag), _ptr(d_db), _stream())
    _check('lcf_fallback', st)
