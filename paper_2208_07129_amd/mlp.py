"""Learned cell-local preconditioner for block CG (state, training and
inference; every step runs in the library's kernels, include/mfmlp.h).

    z = D^{-1} r + sum_e Q_e^T W_e^{1/2} rho_e f_theta(W_e^{1/2} Q_e r / rho_e)

f_theta(x) = W3 relu(W2 relu(W1 x + b1) + b2) + b3 + S x with F = np^3 inputs
and outputs, hidden width 256, ReLU, and a symmetric linear skip S (kept
symmetric by projection after every optimizer step).  BF16 weights on the
matrix cores, FP32 master weights, Adam.  The skip is folded into the last
layer: y = [W3 | S] [h2; x] + b3, one GEMM.  W_e are the partition-of-unity
weights, applied as square roots on both sides so that a symmetric cell map
gives a symmetric preconditioner (with f = 0 it is exactly Jacobi).

Training pairs are generated by the operator (make_local_pairs): errors
confined to cells of one colour of an 8-colouring, so for those cells the
residual restricted to the cell is A_ee e_cell with A_ee the cell block of A,
and the network learns the correction (A_ee^{-1} - D_e^{-1}) of the Jacobi
step on each cell.  Rows of a batch are (cell, column) pairs; activations are
stored feature-major (features x rows).
"""
from __future__ import annotations

import ctypes
import math
from dataclasses import dataclass
from typing import Dict, List, Optional

import numpy as np

from . import mfmv
from .mfmv import _check, _stream_ptr, lib


def _ceil8(n: int) -> int:
    return (n + 7) // 8 * 8


def _host_bf16(a: np.ndarray) -> np.ndarray:
    """BF16 bit patterns (int16) of FP32 values, round to nearest even."""
    u = np.asarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return u.view(np.int16)


@dataclass
class TrainLog:
    steps: int = 0
    loss: List[float] = None
    seconds: float = 0.0


class CellMLP:
    """The network and its optimizer state for one operator (cell size np^3)."""

    def __init__(self, op: mfmv.Operator, hidden: int = 256, seed: int = 0, out_scale: float = 0.0,
                 dscale=None):
        """dscale: the operator diagonal; when given, the network works on the
        diagonally scaled cell problem (inputs D^{-1/2} r, targets D^{1/2} e,
        outputs assembled with D^{-1/2})."""
        import torch
        self.op = op
        self.dscale = dscale
        self.F = (op.p + 1) ** 3
        self.Fp = _ceil8(self.F)
        self.H = hidden
        if hidden % 8:
            raise ValueError("hidden width must be a multiple of 8")
        rng = np.random.default_rng(seed)
        F, Fp, H = self.F, self.Fp, self.H
        W1 = np.zeros((H, Fp), np.float32)
        W1[:, :F] = rng.standard_normal((H, F)) * math.sqrt(2.0 / F)
        W2 = (rng.standard_normal((H, H)) * math.sqrt(2.0 / H)).astype(np.float32)
        W3S = np.zeros((Fp, H + Fp), np.float32)     # [W3 | S]
        W3S[:F, :H] = rng.standard_normal((F, H)) * out_scale * math.sqrt(1.0 / H)
        host = [W1, np.zeros(H, np.float32), W2, np.zeros(H, np.float32), W3S,
                np.zeros(Fp, np.float32)]
        dev = torch.device("cuda")
        self.params = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in host]
        self.grads = [torch.empty_like(p) for p in self.params]
        self.m1 = [torch.zeros_like(p) for p in self.params]
        self.m2 = [torch.zeros_like(p) for p in self.params]
        self.wbf = {i: torch.from_numpy(_host_bf16(host[i])).to(dev) for i in (0, 2, 4)}
        self.step = 0
        self._buf: Dict[str, object] = {}
        self._loss = torch.zeros(1, dtype=torch.float64, device=dev)

    # ------------------------------------------------------------ checkpoints
    _NAMES = ("W1", "b1", "W2", "b2", "W3S", "b3")

    def state(self) -> dict:
        """Host copies of everything training needs to resume: the FP32 master
        weights, their BF16 copies, both Adam moments and the step counter."""
        st = {}
        for name, w, m1, m2 in zip(self._NAMES, self.params, self.m1, self.m2):
            st[name] = w.detach().cpu()
            st["adam_m1." + name] = m1.detach().cpu()
            st["adam_m2." + name] = m2.detach().cpu()
        for i, wb in self.wbf.items():
            st["bf16." + self._NAMES[i]] = wb.detach().cpu()
        return st

    def save(self, path: str) -> None:
        """Write a checkpoint (safetensors: tensors plus the shape metadata and
        step; loading it executes nothing from the file)."""
        from safetensors.torch import save_file
        meta = {"format": "cellmlp-1", "F": str(self.F), "Fp": str(self.Fp), "H": str(self.H),
                "p": str(self.op.p), "step": str(self.step)}
        save_file({k: v.contiguous() for k, v in self.state().items()}, path, metadata=meta)

    def load(self, path: str) -> None:
        """Resume from a checkpoint written by save() for a network of the same
        shape (cell size and hidden width); raises ValueError otherwise."""
        from safetensors import safe_open
        with safe_open(path, framework="pt", device="cpu") as f:
            meta = f.metadata() or {}
            if meta.get("format") != "cellmlp-1":
                raise ValueError(f"{path}: not a cell-network checkpoint")
            for key, want in (("F", self.F), ("Fp", self.Fp), ("H", self.H)):
                if int(meta.get(key, -1)) != want:
                    raise ValueError(f"{path}: {key} = {meta.get(key)}, this network has {want}")
            tensors = {k: f.get_tensor(k) for k in f.keys()}
        for name, w, m1, m2 in zip(self._NAMES, self.params, self.m1, self.m2):
            for dst, key in ((w, name), (m1, "adam_m1." + name), (m2, "adam_m2." + name)):
                src = tensors[key]
                if tuple(src.shape) != tuple(dst.shape) or src.dtype != dst.dtype:
                    raise ValueError(f"{path}: {key} has shape {tuple(src.shape)} {src.dtype}")
                dst.copy_(src)
        for i, wb in self.wbf.items():
            wb.copy_(tensors["bf16." + self._NAMES[i]])
        self.step = int(meta["step"])

    # ------------------------------------------------------------ buffers
    def _buffers(self, k: int):
        """Activation blocks for ncells * k rows, stored with the row count padded
        to a multiple of 8 (padding columns stay zero in inputs, targets and
        output gradients, so they add nothing to the gradients).  HX stacks h2
        (first H rows) over the input x (next Fp rows): the operand of the last
        layer [W3 | S]."""
        import torch
        rows = self.op.ncells * k
        if self._buf.get("rows") != rows:
            dev = torch.device("cuda")
            Fp, H, ld = self.Fp, self.H, _ceil8(rows)
            i16, f32 = torch.int16, torch.float32
            HX = torch.zeros(H + Fp, ld, dtype=i16, device=dev)
            self._buf = dict(
                rows=rows, ld=ld, HX=HX, H2=HX[:H], X0=HX[H:],
                H1=torch.zeros(H, ld, dtype=i16, device=dev),
                Y=torch.zeros(Fp, ld, dtype=f32, device=dev),
                T=torch.zeros(Fp, ld, dtype=f32, device=dev),
                dY=torch.zeros(Fp, ld, dtype=i16, device=dev),
                dH2=torch.zeros(H, ld, dtype=i16, device=dev),
                dH1=torch.zeros(H, ld, dtype=i16, device=dev),
                rho=torch.zeros(ld, dtype=f32, device=dev),
            )
        return self._buf

    # ------------------------------------------------------------ kernels
    @staticmethod
    def _gemm(M, N, K, ta, tb, A, lda, B, ldb, kchunk=0, bias=None, relu=False, mask=None,
              ldmask=0, out_f32=None, ld_f32=0, atomic=False, out_bf16=None, ld_bf16=0, kb=0):
        ptr = (lambda t: None if t is None else t.data_ptr())
        _check(lib().mf_mlp_gemm(M, N, K, int(ta), int(tb), A.data_ptr(), lda, B.data_ptr(), ldb,
                                 kchunk, ptr(bias), int(relu), ptr(mask), ldmask, ptr(out_f32),
                                 ld_f32, int(atomic), ptr(out_bf16), ld_bf16, kb,
                                 _stream_ptr(None)))

    def gather(self, R, E=None, pou_sqrt: bool = False, normalise: bool = True,
               blocked: bool = False):
        """Network inputs (and targets) of every (cell, column) of R (and E);
        normalise=False skips the per-row RMS scaling (rho = 1); blocked=True
        writes them in the cell-blocked layout (block stride Fp k)."""
        b = self._buffers(R.shape[1])
        k = R.shape[1]
        _check(lib().mf_cell_gather(self.op._h, k, R.data_ptr(), R.stride(0),
                                    None if E is None else E.data_ptr(),
                                    0 if E is None else E.stride(0), self.Fp, b["X0"].data_ptr(),
                                    None if E is None else b["T"].data_ptr(),
                                    self.Fp * k if blocked else b["ld"],
                                    b["rho"].data_ptr() if normalise else None, int(pou_sqrt),
                                    None if self.dscale is None else self.dscale.data_ptr(),
                                    int(blocked), _stream_ptr(None)))
        return b

    def _hidden(self, b):
        n, Fp, H = b["ld"], self.Fp, self.H
        _, b1, _, b2, _, _ = self.params
        self._gemm(H, n, Fp, False, False, self.wbf[0], Fp, b["X0"], n, bias=b1, relu=True,
                   out_bf16=b["H1"], ld_bf16=n)
        self._gemm(H, n, H, False, False, self.wbf[2], H, b["H1"], n, bias=b2, relu=True,
                   out_bf16=b["H2"], ld_bf16=n)

    def forward(self, b):
        n, Fp, H = b["ld"], self.Fp, self.H
        b3 = self.params[5]
        self._hidden(b)
        self._gemm(Fp, n, H + Fp, False, False, self.wbf[4], H + Fp, b["HX"], n, bias=b3,
                   out_f32=b["Y"], ld_f32=n)
        return b["Y"]

    def backward(self, b, kchunk: int = 8192):
        """Gradients of the last loss_grad (dY in b['dY']) into self.grads."""
        n, Fp, H = b["ld"], self.Fp, self.H
        gW1, gb1, gW2, gb2, gW3S, gb3 = self.grads
        s = _stream_ptr(None)
        for g in (gW1, gW2, gW3S):
            _check(lib().mf_fill_f32(g.numel(), g.data_ptr(), 0.0, s))
        # last layer [W3 | S] on [h2; x]
        self._gemm(Fp, H + Fp, n, False, True, b["dY"], n, b["HX"], n, kchunk=kchunk,
                   out_f32=gW3S, ld_f32=H + Fp, atomic=True)
        _check(lib().mf_row_sums(Fp, n, b["dY"].data_ptr(), n, gb3.data_ptr(), 0, s))
        self._gemm(H, n, Fp, True, False, self.wbf[4], H + Fp, b["dY"], n, mask=b["H2"],
                   ldmask=n, out_bf16=b["dH2"], ld_bf16=n)
        # layer 2
        self._gemm(H, H, n, False, True, b["dH2"], n, b["H1"], n, kchunk=kchunk,
                   out_f32=gW2, ld_f32=H, atomic=True)
        _check(lib().mf_row_sums(H, n, b["dH2"].data_ptr(), n, gb2.data_ptr(), 0, s))
        self._gemm(H, n, H, True, False, self.wbf[2], H, b["dH2"], n, mask=b["H1"],
                   ldmask=n, out_bf16=b["dH1"], ld_bf16=n)
        # layer 1
        self._gemm(H, Fp, n, False, True, b["dH1"], n, b["X0"], n, kchunk=kchunk,
                   out_f32=gW1, ld_f32=Fp, atomic=True)
        _check(lib().mf_row_sums(H, n, b["dH1"].data_ptr(), n, gb1.data_ptr(), 0, s))

    def loss_grad(self, b, roww=None, scale: Optional[float] = None) -> None:
        """Weighted mean squared error of the last forward against b['T'] (rows
        weighted by roww, mean over the weight sum) and its output gradient."""
        if scale is None:
            scale = 1.0 / b["rows"]
        _check(lib().mf_mse_grad(self.F, self.Fp, b["rows"], b["Y"].data_ptr(), b["T"].data_ptr(),
                                 b["ld"], None if roww is None else roww.data_ptr(),
                                 ctypes.c_float(scale), b["dY"].data_ptr(),
                                 self._loss.data_ptr(), _stream_ptr(None)))

    def _last_layer_grad(self, b, roww=None, scale: Optional[float] = None) -> None:
        """The last layer and loss_grad in one call (b['Y'] is a work array here)."""
        if scale is None:
            scale = 1.0 / b["rows"]
        _check(lib().mf_mlp_loss_grad(self.F, self.Fp, b["ld"], b["rows"], self.H + self.Fp,
                                      self.wbf[4].data_ptr(), self.H + self.Fp, b["HX"].data_ptr(),
                                      self.params[5].data_ptr(), b["T"].data_ptr(), b["ld"],
                                      None if roww is None else roww.data_ptr(),
                                      ctypes.c_float(scale), b["dY"].data_ptr(),
                                      b["Y"].data_ptr(), self._loss.data_ptr(), _stream_ptr(None)))

    def adam(self, lr: float, b1: float = 0.9, b2: float = 0.999, eps: float = 1e-8):
        self.step += 1
        for i, (w, g, m1, m2) in enumerate(zip(self.params, self.grads, self.m1, self.m2)):
            wbf = self.wbf.get(i)
            _check(lib().mf_adam(w.numel(), w.data_ptr(), g.data_ptr(), m1.data_ptr(),
                                 m2.data_ptr(), None if wbf is None else wbf.data_ptr(),
                                 ctypes.c_float(lr), ctypes.c_float(b1), ctypes.c_float(b2),
                                 ctypes.c_float(eps), self.step, _stream_ptr(None)))
        self.project()

    def project(self):
        """Keep the skip block S (columns H.. of the last layer) symmetric."""
        W3S, H = self.params[4], self.H
        ld = self.H + self.Fp
        _check(lib().mf_symmetrize(self.F, W3S[:, H:].data_ptr(), ld,
                                   self.wbf[4][:, H:].data_ptr(), _stream_ptr(None)))

    def train_step(self, R, T_err, lr: float, roww=None, scale: Optional[float] = None) -> float:
        """One Adam step on the pairs (R, T_err) (T_err: the error to predict, in
        the Jacobi-correction form E - D^{-1} R; rows weighted by roww); returns
        the loss before the step."""
        b = self.gather(R, T_err)
        self._hidden(b)
        self._loss.zero_()
        self._last_layer_grad(b, roww, scale)
        self.backward(b)
        self.adam(lr)
        return float(self._loss.item())

    def eval_loss(self, R, T_err, roww=None, scale: Optional[float] = None) -> float:
        b = self.gather(R, T_err)
        self.forward(b)
        self._loss.zero_()
        self.loss_grad(b, roww, scale)
        return float(self._loss.item())

    def precondition(self, R, Z, diag, linear: bool = False) -> None:
        """Z := D^{-1} R + sum_e Q_e^T W_e^{1/2} rho f(W_e^{1/2} Q_e R / rho).
        linear=True keeps only the symmetric skip S (no ReLU branch, no bias):
        a fixed symmetric linear preconditioner, for which the scale rho
        cancels (gathered and assembled without it).  With k a multiple of 8 the
        linear path keeps its activations in the cell-blocked layout, so gather
        and assembly stream whole cells."""
        k = R.shape[1]
        blocked = linear and k % 8 == 0
        Fp, H = self.Fp, self.H
        b = self._buffers(k) if blocked else self.gather(R, pou_sqrt=True, normalise=not linear)
        ld = Fp * k if blocked else b["ld"]
        if blocked:
            _check(lib().mf_cell_linear(self.op._h, k, R.data_ptr(), R.stride(0), Fp,
                                        self.wbf[4][:, H:].data_ptr(), H + Fp, b["X0"].data_ptr(),
                                        b["Y"].data_ptr(), ld, 1,
                                        None if self.dscale is None else self.dscale.data_ptr(),
                                        _stream_ptr(None)))
        elif linear:
            self._gemm(Fp, ld, Fp, False, False, self.wbf[4][:, H:], H + Fp, b["X0"], ld,
                       out_f32=b["Y"], ld_f32=ld)
        else:
            self.forward(b)
        _check(lib().mf_cell_scatter(self.op._h, k, b["Y"].data_ptr(), ld,
                                     None if linear else b["rho"].data_ptr(), diag.data_ptr(),
                                     R.data_ptr(), R.stride(0), Z.data_ptr(), Z.stride(0), 1,
                                     None if self.dscale is None else self.dscale.data_ptr(),
                                     int(blocked), _stream_ptr(None)))

    def floor_skip(self, margin: float = 0.02) -> int:
        """Raise the eigenvalues of the skip block S to at least
        -1 + margin + 2^-8 (||S||_F + sqrt(F)) (mf_skip_floor): then I + S, and
        with it the linear preconditioner, stays positive definite after the BF16
        rounding of the deployed copy.  Returns mf_sym_eig's status (0: done)."""
        import torch
        W3S, H, F = self.params[4], self.H, self.F
        ld = H + self.Fp
        work = torch.empty(int(lib().mf_skip_floor_work(F)), dtype=torch.float64,
                           device=W3S.device)
        st = torch.zeros(1, dtype=torch.int32, device=W3S.device)
        _check(lib().mf_skip_floor(F, W3S[:, H:].data_ptr(), ld, self.wbf[4][:, H:].data_ptr(), ld,
                                   ctypes.c_double(margin), work.data_ptr(), work.numel(),
                                   st.data_ptr(), _stream_ptr(None)))
        return int(st.item())

    def preconditioner(self, diag, linear: bool = True):
        """Preconditioner callable for blockcg.  Default: the trained symmetric
        linear part S on top of Jacobi, a fixed cell-wise operator; after
        floor_skip() it is symmetric positive definite up to the BF16 rounding
        of its input, so block PCG keeps its short recurrence.  linear=False uses
        the whole network (nonlinear: flexible iteration, less robust)."""
        def M(R, Z):
            self.precondition(R, Z, diag, linear)
            return Z
        return M


# ---------------------------------------------------------------- training data
def make_pairs(op: mfmv.Operator, diag, k: int, seed: int, smooth_steps: int, omega: float = 0.6):
    """(R, T) with E random U[-1, 1] columns smoothed by `smooth_steps` damped
    Jacobi sweeps on the error (e <- e - omega D^{-1} A e), R = A E and the
    Jacobi-correction target T = E - D^{-1} R.  All steps are library calls."""
    import torch
    rng = np.random.default_rng(seed)
    E = torch.from_numpy(rng.uniform(-1.0, 1.0, (op.ndofs, k))).cuda()
    AE = torch.empty_like(E)
    for _ in range(smooth_steps):
        op.apply(E, AE)
        mfmv.jacobi(diag, AE, AE)
        mfmv.axpby(-omega, AE, 1.0, E)
    R = torch.empty_like(E)
    op.apply(E, R)
    T = torch.empty_like(E)
    mfmv.jacobi(diag, R, T)
    mfmv.axpby(1.0, E, -1.0, T)   # T = E - D^{-1} R
    return R, T, E


def cell_colors(op: mfmv.Operator) -> np.ndarray:
    """Colour 0..7 of every cell from the parities of its coordinates, so cells of
    one colour share no node; -1 for cells left out (the last layer of a periodic
    direction with an odd cell count, which wraps onto the first)."""
    n = [int(v) for v in op.mesh.n]
    cz, cy, cx = np.meshgrid(np.arange(n[2]), np.arange(n[1]), np.arange(n[0]), indexing="ij")
    col = (cx % 2) + 2 * (cy % 2) + 4 * (cz % 2)
    if op.mesh.bc == 2:  # periodic
        for c, nd in zip((cx, cy, cz), n):
            if nd % 2 == 1 and nd > 1:
                col = np.where(c == nd - 1, -1, col)
            if nd == 1:
                col = np.full_like(col, -1)
    return col.ravel()


def _host_cell_nodes(op: mfmv.Operator) -> np.ndarray:
    """Global node numbers (E x np^3, -1 constrained) in the library's numbering:
    node (gx, gy, gz) -> gx + Nx (gy + Ny gz), local index i1 + np (i2 + np i3)."""
    p, n = op.p, [int(v) for v in op.mesh.n]
    per = op.mesh.bc == 2
    N = [nd * p + (0 if per else 1) for nd in n]
    cz, cy, cx = np.meshgrid(np.arange(n[2]), np.arange(n[1]), np.arange(n[0]), indexing="ij")
    i3, i2, i1 = np.meshgrid(np.arange(p + 1), np.arange(p + 1), np.arange(p + 1), indexing="ij")
    g = [(c.ravel()[:, None] * p + i.ravel()[None, :]) for c, i in ((cx, i1), (cy, i2), (cz, i3))]
    if per:
        g = [gd % Nd for gd, Nd in zip(g, N)]
    node = g[0] + N[0] * (g[1] + N[1] * g[2])
    if op.mesh.bc == 1:  # zero Dirichlet
        bnd = np.zeros_like(node, dtype=bool)
        for gd, Nd in zip(g, N):
            bnd |= (gd == 0) | (gd == Nd - 1)
        node = np.where(bnd, -1, node)
    return node


def make_local_pairs(op: mfmv.Operator, diag, k: int, seed: int, smooth_frac: float = 0.5):
    """Pairs for which the local problem is exact: column j carries an error
    confined to the cells of colour j % 8 (random values, part of them plus a
    random low-degree polynomial over the cell), so for those cells the
    operator's residual restricted to the cell is A_ee e_cell with A_ee the
    cell block of A.  Returns (R, T, roww, scale) with T = E - D^{-1} R, row
    weights 1 on the (cell, column) rows of matching colour, 0 elsewhere."""
    import torch
    rng = np.random.default_rng(seed)
    nodes = _host_cell_nodes(op)
    colors = cell_colors(op)
    np1 = op.p + 1
    xi = np.linspace(-1.0, 1.0, np1)
    P = np.stack([np.ones(np1), xi, 1.5 * xi * xi - 0.5])   # degree 0, 1, 2
    E = np.zeros((op.ndofs, k))
    roww = np.zeros(op.ncells * k, np.float32)
    for j in range(k):
        cells = np.nonzero(colors == j % 8)[0]
        if cells.size == 0:
            continue
        vals = rng.uniform(-1.0, 1.0, (cells.size, np1 ** 3))
        smooth = rng.random(cells.size) < smooth_frac
        if smooth.any():
            c = rng.standard_normal((int(smooth.sum()), 3, 3, 3))
            poly = np.einsum("sabc,ak,bj,ci->sijk", c, P, P, P).reshape(-1, np1 ** 3)
            vals[smooth] = 0.3 * vals[smooth] + poly
        nd = nodes[cells]
        live = nd >= 0
        E[nd[live], j] = vals[live]
        roww[cells * k + j] = 1.0
    Ed = torch.from_numpy(E).cuda()
    R = torch.empty_like(Ed)
    op.apply(Ed, R)
    T = torch.empty_like(Ed)
    mfmv.jacobi(diag, R, T)
    mfmv.axpby(1.0, Ed, -1.0, T)   # T = E - D^{-1} R
    w = torch.from_numpy(roww).cuda()
    return R, T, w, 1.0 / max(float(roww.sum()), 1.0)


def train(net: CellMLP, diag, steps: int, k: int = 16, lr: float = 3e-3, seed: int = 0,
          refresh: int = 1, log: Optional[list] = None, checkpoint: Optional[str] = None,
          every: int = 0) -> list:
    """Adam on fresh local pairs from the operator (make_local_pairs), a new
    pair block every `refresh` steps, until the network has taken `steps` steps
    in total: a network restored with net.load() continues from its step
    counter with the pairs it would have drawn next, so an interrupted run
    resumes where its last checkpoint left it.  With `checkpoint`, the state is
    saved there every `every` steps (if > 0) and at the end."""
    losses = [] if log is None else log
    pairs = None
    for s in range(net.step, steps):
        if pairs is None or s % refresh == 0:
            s0 = s - s % refresh
            pairs = make_local_pairs(net.op, diag, k, seed * 100003 + s0)
        R, T, w, sc = pairs
        losses.append(net.train_step(R, T, lr, w, sc))
        if checkpoint and every > 0 and net.step % every == 0:
            net.save(checkpoint)
    if checkpoint:
        net.save(checkpoint)
    return losses


def local_fit(net: CellMLP, diag, k: int = 16, seed: int = 999) -> float:
    """Held-out relative squared error of the learned correction on local pairs:
    sum ||f(x) - t||^2 / sum ||t||^2 over the rows that count (0: exact cell-block
    inverse; 1: no better than the Jacobi step)."""
    import torch
    R, T, w, sc = make_local_pairs(net.op, diag, k, seed)
    err = net.eval_loss(R, T, w, sc)
    b = net._buffers(k)
    Y = b["Y"]
    keep = Y.clone()
    _check(lib().mf_fill_f32(Y.numel(), Y.data_ptr(), 0.0, _stream_ptr(None)))
    net._loss.zero_()
    net.loss_grad(b, w, sc)
    ref = float(net._loss.item())
    Y.copy_(keep)
    return err / max(ref, 1e-300)


def a_norm_error(op: mfmv.Operator, E, Z):
    """Per column ||E - Z||_A^2 (FP64 apply and library dot products)."""
    import torch
    D = torch.empty_like(E)
    mfmv.axpby(1.0, E, 0.0, D)
    mfmv.axpby(-1.0, Z, 1.0, D)
    AD = torch.empty_like(D)
    op.apply(D, AD)
    return mfmv.col_dots(D, AD).cpu().numpy()


def judge(net: CellMLP, diag, k: int = 16, seed: int = 12345, depths=(0, 2, 8),
          linear: bool = True) -> dict:
    """Held-out check of the learned step against the Jacobi step: the A-norm
    of the error left by one application, z = M(r) for r = A e, averaged over
    columns and smoothing depths.  ratio < 1: the network improves on Jacobi."""
    import torch
    num, den = 0.0, 0.0
    for i, d in enumerate(depths):
        R, _, E = make_pairs(net.op, diag, k, seed + i, d)
        Zl = torch.empty_like(R)
        net.precondition(R, Zl, diag, linear)
        Zj = torch.empty_like(R)
        mfmv.jacobi(diag, R, Zj)
        # best scalar multiple of each step (CG rescales directions anyway)
        for Z, acc in ((Zl, "l"), (Zj, "j")):
            AZ = torch.empty_like(Z)
            net.op.apply(Z, AZ)
            zaz = mfmv.col_dots(Z, AZ).cpu().numpy()
            zae = mfmv.col_dots(AZ, E).cpu().numpy()
            AE = torch.empty_like(E)
            net.op.apply(E, AE)
            eae = mfmv.col_dots(E, AE).cpu().numpy()
            left = np.mean(1.0 - zae ** 2 / np.maximum(zaz * eae, 1e-300))
            if acc == "l":
                num += left
            else:
                den += left
    return {"learned": num / len(depths), "jacobi": den / len(depths),
            "ratio": num / max(den, 1e-300)}
