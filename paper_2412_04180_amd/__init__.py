"""Thin Python binding of libskim (gfx950): argument marshalling only.

Every step of the hot path runs inside the HIP library behind the C ABI of
include/skim.h.  torch is used for device memory and the stream.  There is no
CPU fallback: importing works anywhere, but creating a context without the
built library or without a GPU raises.
"""
from __future__ import annotations

import ctypes as C
import os

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libskim.so")

SKIM_OK = 0
STATUS_NAMES = {0: "SKIM_OK", -1: "SKIM_ERR_ARG", -2: "SKIM_ERR_SHAPE", -3: "SKIM_ERR_BUDGET",
                -4: "SKIM_ERR_WORKSPACE", -5: "SKIM_ERR_HIP", -6: "SKIM_ERR_NONFINITE"}
MAX_M = 32768
PACK_STATIC_MAX_ROWS = 65536

EXPORTS = ["skim_create", "skim_destroy", "skim_last_error", "skim_workspace_bytes", "skim_set_workspace",
           "skim_profile_enable", "skim_profile_last", "skim_validate_enable",
           "skim_error_table", "skim_error_table_lfull", "skim_cluster_rows", "skim_select_allocated", "skim_greedy_allocate", "skim_greedy_allocate_device",
           "skim_dp_allocate_scratch_bytes", "skim_dp_allocate", "skim_kmeans_optimal_scratch_bytes", "skim_kmeans_optimal",
           "skim_packed_words", "skim_codebook_entries", "skim_pack", "skim_pack_static", "skim_layer_loss", "skim_scale_step", "skim_train_scale", "skim_unpack", "skim_dequant_matvec", "skim_dequant_matvec_f32", "skim_hessian_workspace_bytes", "skim_hessian_from_activations", "skim_hessian_from_activations_scratch"]


class SkimError(RuntimeError):
    def __init__(self, status, text):
        super().__init__(f"{STATUS_NAMES.get(status, status)}: {text}")
        self.status = status


class AdamOpts(C.Structure):
    _fields_ = [("lr0", C.c_float), ("beta1", C.c_float), ("beta2", C.c_float), ("eps", C.c_float),
                ("decay", C.c_float), ("decay_every", C.c_int32)]


_lib = None


def load_library():
    """dlopen the in-tree libskim.so; raises when it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2412_04180_amd._build` "
                               "(there is no fallback path)")
        # torch owns device memory and streams: load it first so that the library binds to the
        # HIP runtime torch has already loaded (one runtime per process)
        import torch  # noqa: F401

        lib = C.CDLL(LIB_PATH)
        vp, i64, i32, dbl = C.c_void_p, C.c_int64, C.c_int, C.c_double
        lib.skim_create.argtypes = [C.POINTER(vp), i32, vp]
        lib.skim_destroy.argtypes = [vp]
        lib.skim_last_error.argtypes = [vp]
        lib.skim_last_error.restype = C.c_char_p
        lib.skim_workspace_bytes.argtypes = [i64, i64]
        lib.skim_workspace_bytes.restype = C.c_size_t
        lib.skim_set_workspace.argtypes = [vp, vp, C.c_size_t]
        lib.skim_profile_enable.argtypes = [vp, i32]
        lib.skim_validate_enable.argtypes = [vp, i32]
        lib.skim_profile_last.argtypes = [vp, C.POINTER(C.c_float), C.POINTER(C.c_float)]
        lib.skim_error_table.argtypes = [vp, vp, vp, vp, i64, i64, i64, i32, i32, i32, vp, vp, vp]
        lib.skim_error_table_lfull.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, i32, i32, i32, vp, vp, vp, vp, vp]
        lib.skim_cluster_rows.argtypes = [vp, vp, vp, vp, i64, i64, i64, vp, i32, vp, vp, vp, vp]
        lib.skim_select_allocated.argtypes = [vp, i64, i32, i32, vp, vp, vp, vp, vp, vp, vp]
        lib.skim_greedy_allocate.argtypes = [vp, vp, i64, i32, i32, dbl, vp, vp, vp]
        lib.skim_greedy_allocate_device.argtypes = [vp, vp, i64, i32, i32, dbl, vp, vp]
        lib.skim_dp_allocate_scratch_bytes.argtypes = [i64, i32, i32, dbl]
        lib.skim_dp_allocate_scratch_bytes.restype = C.c_size_t
        lib.skim_dp_allocate.argtypes = [vp, vp, i64, i32, i32, dbl, vp, vp, vp, C.c_size_t]
        lib.skim_kmeans_optimal_scratch_bytes.argtypes = [i64, i64]
        lib.skim_kmeans_optimal_scratch_bytes.restype = C.c_size_t
        lib.skim_kmeans_optimal.argtypes = [vp, vp, vp, vp, i64, i64, i64, i32, i32, vp, vp, C.c_size_t]
        lib.skim_packed_words.argtypes = [vp, i64, i64]
        lib.skim_packed_words.restype = i64
        lib.skim_codebook_entries.argtypes = [vp, i64]
        lib.skim_codebook_entries.restype = i64
        lib.skim_pack.argtypes = [vp, vp, vp, i64, i64, i64, vp, vp, vp, vp, vp, vp, vp, vp]
        lib.skim_pack_static.argtypes = [vp, vp, vp, i64, i64, i64, vp, vp, vp, vp, vp, vp, vp, vp]
        lib.skim_layer_loss.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, vp, vp, vp]
        lib.skim_scale_step.argtypes = [vp, vp, vp, vp, i64, i64, i64, vp, vp, vp, vp, i64, C.POINTER(AdamOpts), vp, vp]
        lib.skim_hessian_workspace_bytes.argtypes = [vp, i64, i64]
        lib.skim_hessian_workspace_bytes.restype = C.c_size_t
        lib.skim_hessian_from_activations.argtypes = [vp, vp, i64, i64, vp]
        lib.skim_hessian_from_activations_scratch.argtypes = [vp, vp, i64, i64, vp, vp, C.c_size_t]
        lib.skim_unpack.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, vp]
        lib.skim_dequant_matvec.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, vp, vp]
        lib.skim_dequant_matvec_f32.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, vp, vp]
        lib.skim_train_scale.argtypes = [vp, vp, vp, vp, i64, i64, i64, vp, i32, i32, i32, i64, C.POINTER(AdamOpts),
                                         vp, vp, vp, vp, vp, vp]
        _lib = lib
    return _lib


def _dp(t):
    """Device pointer of a torch tensor (None -> NULL)."""
    return None if t is None else C.c_void_p(t.data_ptr())


def greedy_allocate(E, avg_bits, bmin=1, bmax=4, row_cost=None):
    """skim_greedy_allocate on host arrays.  Returns (bits uint8[n], spent, budget)."""
    lib = load_library()
    E = np.ascontiguousarray(E, dtype=np.float64)
    n = E.shape[0]
    if E.ndim != 2 or E.shape[1] != bmax - bmin + 1:
        raise ValueError("E must be n x (bmax-bmin+1)")
    cost = None if row_cost is None else np.ascontiguousarray(row_cost, dtype=np.int64)
    bits = np.empty(n, np.uint8)
    spent, budget = C.c_int64(0), C.c_int64(0)
    st = lib.skim_greedy_allocate(E.ctypes.data_as(C.c_void_p), None if cost is None else cost.ctypes.data_as(C.c_void_p),
                                  n, bmin, bmax, float(avg_bits), bits.ctypes.data_as(C.c_void_p),
                                  C.cast(C.byref(spent), C.c_void_p), C.cast(C.byref(budget), C.c_void_p))
    if st != SKIM_OK:
        raise SkimError(st, "skim_greedy_allocate")
    return bits, spent.value, budget.value


def packed_words(bits, m):
    bits = np.ascontiguousarray(bits, dtype=np.uint8)
    return int(load_library().skim_packed_words(bits.ctypes.data_as(C.c_void_p), len(bits), m))


def codebook_entries(bits):
    bits = np.ascontiguousarray(bits, dtype=np.uint8)
    return int(load_library().skim_codebook_entries(bits.ctypes.data_as(C.c_void_p), len(bits)))


class Context:
    """One skim_ctx bound to a torch device and stream."""

    def __init__(self, device=0, stream=None):
        import torch

        self.torch = torch
        self.lib = load_library()
        if not torch.cuda.is_available():
            raise RuntimeError("no GPU visible: the SKIM hot path has no CPU fallback")
        self.device = torch.device("cuda", device)
        torch.cuda.set_device(self.device)
        self.stream = stream if stream is not None else torch.cuda.current_stream(self.device)
        h = C.c_void_p()
        st = self.lib.skim_create(C.byref(h), device, C.c_void_p(self.stream.cuda_stream))
        if st != SKIM_OK:
            raise SkimError(st, self.lib.skim_last_error(None).decode())
        self.h = h
        self._ws = None
        self._hessian_blocks = []

    def close(self):
        if getattr(self, "h", None):
            self.lib.skim_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, st):
        if st != SKIM_OK:
            raise SkimError(st, self.lib.skim_last_error(self.h).decode())

    def workspace_bytes(self, n, m):
        return int(self.lib.skim_workspace_bytes(n, m))

    def ensure_workspace(self, n, m):
        need = self.workspace_bytes(n, m)
        if self._ws is None or self._ws.numel() < need:
            # allocated on the context's stream: torch's allocator then ties the lifetime of the old block to
            # the work already queued on that stream
            with self.torch.cuda.stream(self.stream):
                self._ws = self.torch.empty(need, dtype=self.torch.uint8, device=self.device)
            self._check(self.lib.skim_set_workspace(self.h, _dp(self._ws), need))

    def validate_enable(self, on=True):
        """Make the clustering calls check W, S and alpha first (they then synchronise and raise SkimError with
        status SKIM_ERR_NONFINITE on a value the method is not defined on)."""
        self._check(self.lib.skim_validate_enable(self.h, 1 if on else 0))

    def profile_enable(self, on=True):
        self._check(self.lib.skim_profile_enable(self.h, 1 if on else 0))

    def profile_last(self):
        """(sort_ms, lloyd_ms) of the last clustering call made with profiling on (synchronises)."""
        a, b = C.c_float(0), C.c_float(0)
        self._check(self.lib.skim_profile_last(self.h, C.byref(a), C.byref(b)))
        return a.value, b.value

    def empty(self, shape, dtype):
        with self.torch.cuda.stream(self.stream):     # outputs belong to the stream the kernels run on
            return self.torch.empty(shape, dtype=dtype, device=self.device)

    # -- clustering -----------------------------------------------------------
    def error_table(self, W, S, alpha=None, bmin=1, bmax=4, iters=30, want_centroids=True, want_upper=True,
                    out=None):
        """W, S: float32 device tensors n x m (row stride = W.stride(0)).  Returns dict of device tensors."""
        t = self.torch
        n, m = W.shape
        assert W.dtype == t.float32 and S.dtype == t.float32 and W.stride(1) == 1 and S.stride() == W.stride()
        nb = bmax - bmin + 1
        stride = (2 << bmax) - (1 << bmin)
        if out is None:
            out = dict(E=self.empty((n, nb), t.float64),
                       centroids_all=self.empty((n, stride), t.float64) if want_centroids else None,
                       upper_all=self.empty((n, stride), t.float32) if want_upper else None)
        self.ensure_workspace(n, m)
        self._check(self.lib.skim_error_table(self.h, _dp(W), _dp(S), _dp(alpha), n, m, W.stride(0), bmin, bmax,
                                              iters, _dp(out["E"]), _dp(out.get("centroids_all")),
                                              _dp(out.get("upper_all"))))
        return out

    def error_table_lfull(self, W, S, H, alpha=None, bmin=1, bmax=4, iters=30, out=None):
        """Error table with the layer-wise (L-full) error of every clustering; H: float32 device m x m."""
        t = self.torch
        n, m = W.shape
        assert W.dtype == t.float32 and S.dtype == t.float32 and W.stride(1) == 1 and S.stride() == W.stride()
        assert H.dtype == t.float32 and H.shape == (m, m) and H.is_contiguous()
        nb = bmax - bmin + 1
        stride = (2 << bmax) - (1 << bmin)
        if out is None:
            out = dict(E_full=self.empty((n, nb), t.float64), E=self.empty((n, nb), t.float64),
                       centroids_all=self.empty((n, stride), t.float64), upper_all=self.empty((n, stride), t.float32),
                       labels_work=self.empty((n, m), t.uint8))
        self.ensure_workspace(n, m)
        self._check(self.lib.skim_error_table_lfull(self.h, _dp(W), _dp(S), _dp(alpha), _dp(H), n, m, W.stride(0),
                                                    bmin, bmax, iters, _dp(out["E_full"]), _dp(out.get("E")),
                                                    _dp(out["centroids_all"]), _dp(out["upper_all"]),
                                                    _dp(out["labels_work"])))
        return out

    def cluster_rows(self, W, S, bits, alpha=None, iters=30, want_labels=True, out=None):
        t = self.torch
        n, m = W.shape
        assert W.dtype == t.float32 and S.dtype == t.float32 and W.stride(1) == 1 and S.stride() == W.stride()
        assert bits.dtype == t.uint8 and bits.numel() == n
        self.ensure_workspace(n, m)
        if out is None:
            out = dict(labels=self.empty((n, m), t.uint8) if want_labels else None,
                       centroids=self.empty((n, 16), t.float64), upper=self.empty((n, 16), t.float32),
                       err=self.empty((n,), t.float64))
        self._check(self.lib.skim_cluster_rows(self.h, _dp(W), _dp(S), _dp(alpha), n, m, W.stride(0), _dp(bits),
                                               iters, _dp(out.get("labels")), _dp(out["centroids"]),
                                               _dp(out.get("upper")), _dp(out["err"])))
        return out

    def select_allocated(self, bits, table, bmin=1, bmax=4, out=None):
        t = self.torch
        n = bits.numel()
        if out is not None:
            cent, upper, err = out["centroids"], out.get("upper"), out.get("err")
        else:
            cent = self.empty((n, 16), t.float64)
            upper = self.empty((n, 16), t.float32) if table.get("upper_all") is not None else None
            err = self.empty((n,), t.float64)
        self._check(self.lib.skim_select_allocated(self.h, n, bmin, bmax, _dp(bits), _dp(table["E"]),
                                                   _dp(table["centroids_all"]), _dp(table.get("upper_all")),
                                                   _dp(cent), _dp(upper), _dp(err)))
        return dict(centroids=cent, upper=upper, err=err)

    # -- packing --------------------------------------------------------------
    def greedy_allocate_device(self, E, avg_bits, bmin=1, bmax=4, out=None):
        """Alg. 1 with unit costs on the device.  Returns dict(bits uint8[n], info int64[10]) of device tensors."""
        t = self.torch
        n = E.shape[0]
        assert E.dtype == t.float64 and E.is_contiguous() and E.shape[1] == bmax - bmin + 1
        if out is None:
            out = dict(bits=self.empty((n,), t.uint8), info=self.empty((10,), t.int64))
        self.ensure_workspace(n, 16)
        self._check(self.lib.skim_greedy_allocate_device(self.h, _dp(E), n, bmin, bmax, float(avg_bits),
                                                         _dp(out["bits"]), _dp(out["info"])))
        return out

    def kmeans_optimal(self, W, S, alpha=None, bmin=1, bmax=4):
        """Least clustering error any assignment of each row to at most 2^b clusters can have (exact interval
        dynamic programme on the sorted row).  Returns a device float64 tensor n x (bmax-bmin+1)."""
        t = self.torch
        n, m = W.shape
        assert W.dtype == t.float32 and S.dtype == t.float32 and W.stride(1) == 1 and S.stride() == W.stride()
        self.ensure_workspace(n, m)
        need = self.lib.skim_kmeans_optimal_scratch_bytes(n, m)
        scratch = self.empty((max(need, 256),), t.uint8)
        E = self.empty((n, bmax - bmin + 1), t.float64)
        self._check(self.lib.skim_kmeans_optimal(self.h, _dp(W), _dp(S), _dp(alpha), n, m, W.stride(0), bmin, bmax,
                                                 _dp(E), _dp(scratch), need))
        self._keep = scratch    # the kernels run asynchronously
        return E

    def dp_allocate(self, E, avg_bits, bmin=1, bmax=4):
        """The exact optimum of the allocation problem (knapsack dynamic programme, unit costs) on the device.
        Returns dict(bits uint8[n], info float64[3] = total error, bits spent, budget) of device tensors."""
        t = self.torch
        n = E.shape[0]
        assert E.dtype == t.float64 and E.is_contiguous() and E.shape[1] == bmax - bmin + 1
        need = self.lib.skim_dp_allocate_scratch_bytes(n, bmin, bmax, float(avg_bits))
        if need == 0:
            raise SkimError(-3, "skim_dp_allocate: bit range or budget not representable")
        scratch = self.empty((need,), t.uint8)
        out = dict(bits=self.empty((n,), t.uint8), info=self.empty((3,), t.float64))
        self._check(self.lib.skim_dp_allocate(self.h, _dp(E), n, bmin, bmax, float(avg_bits), _dp(out["bits"]),
                                              _dp(out["info"]), _dp(scratch), need))
        out["_scratch"] = scratch   # the kernels run asynchronously: the buffer lives as long as the result
        return out

    def pack(self, W, bits, centroids, upper, alpha=None, want_dW=False, bits_host=None, max_size=False, out=None):
        """bits: device uint8[n].  bits_host (numpy) sizes the outputs; copied from the device when omitted.
        max_size: size the outputs for 4 bits in every row instead (no copy of bits to the host; the used part
        ends at group_word_offset[5] words)."""
        t = self.torch
        n, m = W.shape
        if out is not None:
            self.ensure_workspace(n, m)
            self._check(self.lib.skim_pack(self.h, _dp(W), _dp(alpha), n, m, W.stride(0), _dp(bits), _dp(centroids),
                                           _dp(upper), _dp(out["codes"]), _dp(out["group_word_offset"]),
                                           _dp(out["row_perm"]), _dp(out["codebooks"]), _dp(out.get("dW"))))
            return out
        if max_size:
            nwords, ncb = n * ((m * 4 + 31) // 32), n * 16
        else:
            if bits_host is None:
                bits_host = bits.cpu().numpy()
            nwords = packed_words(bits_host, m)
            ncb = codebook_entries(bits_host)
        if nwords < 0 or ncb < 0:
            raise ValueError("bits must be in 1..4")
        self.ensure_workspace(n, m)
        codes = self.empty((nwords,), t.int32)
        gwo = self.empty((6,), t.int64)
        perm = self.empty((n,), t.int32)
        cbs = self.empty((ncb,), t.int16)
        dW = self.empty((n, m), t.float32) if want_dW else None
        self._check(self.lib.skim_pack(self.h, _dp(W), _dp(alpha), n, m, W.stride(0), _dp(bits), _dp(centroids),
                                       _dp(upper), _dp(codes), _dp(gwo), _dp(perm), _dp(cbs), _dp(dW)))
        return dict(codes=codes, group_word_offset=gwo, row_perm=perm, codebooks=cbs, dW=dW)

    def pack_static(self, W, alpha, bits, centroids, upper, out):
        """skim_pack_static: the variant of pack that neither allocates nor uses the workspace.  Every output is
        the caller's: out = dict(codes, group_word_offset, row_perm, codebooks[, dW]) of device tensors."""
        n, m = W.shape
        self._check(self.lib.skim_pack_static(self.h, _dp(W), _dp(alpha), n, m, W.stride(0), _dp(bits),
                                              _dp(centroids), _dp(upper), _dp(out["codes"]),
                                              _dp(out["group_word_offset"]), _dp(out["row_perm"]),
                                              _dp(out["codebooks"]), _dp(out.get("dW"))))
        return out

    # -- scaling vector -------------------------------------------------------
    def layer_loss(self, W, S, H, labels, alpha=None, want_row_loss=True):
        t = self.torch
        n, m = W.shape
        self.ensure_workspace(n, m)
        loss = self.empty((1,), t.float64)
        row_loss = self.empty((n,), t.float64) if want_row_loss else None
        self._check(self.lib.skim_layer_loss(self.h, _dp(W), _dp(S), _dp(alpha), _dp(H), n, m, W.stride(0),
                                             _dp(labels), _dp(loss), _dp(row_loss)))
        return dict(loss=loss, row_loss=row_loss)

    def _hessian_scratch(self, need):
        """Scratch of the Hessian: not the workspace, which captured calls may hold (as they may hold a block of this one:
        a block that has become too small is kept until the context goes; sizes double, so all blocks together stay below
        twice the last).  None while the stream is captured, or where the card has no room: the call then runs without."""
        t = self.torch
        blocks = self._hessian_blocks
        if blocks and blocks[-1].numel() >= need:
            return blocks[-1]
        with t.cuda.stream(self.stream):
            if need == 0 or t.cuda.is_current_stream_capturing():
                return None
            try:
                blocks.append(t.empty(max(need, 2 * blocks[-1].numel() if blocks else 0), dtype=t.uint8, device=self.device))
            except t.cuda.OutOfMemoryError:
                return None
        return blocks[-1]

    def hessian_from_activations(self, X_bf16, out=None):
        """H = X^T X / N for X: device tensor N x m of dtype bfloat16 (or its int16/uint16 bit patterns)."""
        N, m = X_bf16.shape
        assert X_bf16.is_contiguous() and X_bf16.element_size() == 2
        H = out if out is not None else self.empty((m, m), self.torch.float32)
        scratch = self._hessian_scratch(int(self.lib.skim_hessian_workspace_bytes(self.h, N, m)))
        self._check(self.lib.skim_hessian_from_activations_scratch(self.h, _dp(X_bf16), N, m, _dp(H), _dp(scratch),
                                                                   0 if scratch is None else scratch.numel()))
        return H

    def unpack(self, pk, m, alpha=None):
        """Dense float32 n x m matrix of the packed model `pk` (the dict Context.pack returns)."""
        n = pk["row_perm"].numel()
        Wq = self.empty((n, m), self.torch.float32)
        self._check(self.lib.skim_unpack(self.h, _dp(pk["codes"]), _dp(pk["group_word_offset"]), _dp(pk["row_perm"]),
                                         _dp(pk["codebooks"]), _dp(alpha), n, m, _dp(Wq)))
        return Wq

    def dequant_matvec(self, pk, m, x, alpha=None, out=None):
        """y = Wq x for the packed model `pk`; y float64[n] in original row order."""
        n = pk["row_perm"].numel()
        y = out if out is not None else self.empty((n,), self.torch.float64)
        self._check(self.lib.skim_dequant_matvec(self.h, _dp(pk["codes"]), _dp(pk["group_word_offset"]),
                                                 _dp(pk["row_perm"]), _dp(pk["codebooks"]), _dp(alpha), n, m,
                                                 _dp(x), _dp(y)))
        return y

    def dequant_matvec_f32(self, pk, m, x, alpha=None, out=None):
        """y = Wq x for the packed model `pk` in float32 arithmetic; y float32[n] in original row order."""
        n = pk["row_perm"].numel()
        y = out if out is not None else self.empty((n,), self.torch.float32)
        self._check(self.lib.skim_dequant_matvec_f32(self.h, _dp(pk["codes"]), _dp(pk["group_word_offset"]),
                                                     _dp(pk["row_perm"]), _dp(pk["codebooks"]), _dp(alpha), n, m,
                                                     _dp(x), _dp(y)))
        return y

    def train_scale(self, W, S, H, bits, alpha, adam_m, adam_v, steps=120, outer=1, t0=1, kmeans_iters=30, opts=None):
        """Alg. 2 as one call; alpha, adam_m, adam_v are updated in place.  Returns labels, centroids, loss_trace."""
        t = self.torch
        n, m = W.shape
        self.ensure_workspace(n, m)
        o = opts if opts is not None else AdamOpts(0.01, 0.9, 0.999, 1e-8, 0.5, 40)
        out = dict(labels=self.empty((n, m), t.uint8), centroids=self.empty((n, 16), t.float64),
                   loss_trace=self.empty((outer * steps + 1,), t.float64))
        self._check(self.lib.skim_train_scale(self.h, _dp(W), _dp(S), _dp(H), n, m, W.stride(0), _dp(bits),
                                              int(kmeans_iters), int(outer), int(steps), int(t0), C.byref(o),
                                              _dp(alpha), _dp(adam_m), _dp(adam_v), _dp(out["labels"]),
                                              _dp(out["centroids"]), _dp(out["loss_trace"])))
        return out

    def scale_step(self, W, S, H, labels, alpha, adam_m, adam_v, t_step, opts=None, want_grad=True):
        t = self.torch
        n, m = W.shape
        self.ensure_workspace(n, m)
        o = opts if opts is not None else AdamOpts(0.01, 0.9, 0.999, 1e-8, 0.5, 40)
        loss = self.empty((1,), t.float64)
        grad = self.empty((m,), t.float32) if want_grad else None
        self._check(self.lib.skim_scale_step(self.h, _dp(W), _dp(S), _dp(H), n, m, W.stride(0), _dp(labels),
                                             _dp(alpha), _dp(adam_m), _dp(adam_v), int(t_step), C.byref(o),
                                             _dp(loss), _dp(grad)))
        return dict(loss_before=loss, grad=grad)
