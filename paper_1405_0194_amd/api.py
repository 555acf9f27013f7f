"""Density matrices of sparse pencils given as ordinary sparse matrices.

    G, GE, tr = density_matrix(H, S, mu, beta, P, outputs=("rho", "E"))

H and S are torch sparse tensors (COO, CSR or CSC, on any device), scipy
sparse matrices or dense arrays; real symmetric, or complex Hermitian (then
the path is the L D U factorization and two-sided selected inversion and the
results are complex).  Only their lower triangles are read: an entry given in
one triangle only is mirrored (conjugated for complex input).  The union of
the two patterns is the pattern of the problem (Sec. II.B: the selected
elements are those of H and S).

This module marshals data: it converts the input once per call to the lower
triangle in CSC, keeps one symbolic analysis per pattern (the analysis is
reused across SCF steps, Sec. II.B) with its factor and workspace buffers,
and returns the pole-expanded matrices (eqs. gammapole, gammaF) as torch
sparse CSC tensors of the lower triangle on the device, with the traces
Tr(G S), Tr(G H) (eq. Nmu and the band energy), Tr(G^E S), the free energy
Tr(G^F S) + mu N and N'(mu) = Tr(G^d S) (Sec. II.C) for the sets asked for.
Every numerical step runs in the HIP library.
"""
import contextlib
import hashlib
import threading

import numpy as np

from . import binding as B

SETS = ("rho", "E", "F", "d")


def _as_coo(M):
    """(n, rows, cols, values) of a square matrix on the host."""
    import scipy.sparse as sp
    try:
        import torch
    except ImportError:          # pragma: no cover
        torch = None
    if torch is not None and isinstance(M, torch.Tensor):
        if M.layout in (torch.sparse_csr, torch.sparse_csc, torch.sparse_bsr, torch.sparse_bsc):
            M = M.to_sparse_coo()
        if M.layout == torch.sparse_coo:
            M = M.coalesce()
            idx = M.indices().cpu().numpy()
            vals = M.values().cpu().numpy()
            return int(M.shape[0]), idx[0].astype(np.int64), idx[1].astype(np.int64), vals, tuple(M.shape)
        M = M.cpu().numpy()
    if sp.issparse(M):
        c = M.tocoo()
        c.sum_duplicates()
        return int(c.shape[0]), c.row.astype(np.int64), c.col.astype(np.int64), c.data, c.shape
    a = np.asarray(M)
    r, c = np.nonzero(a)
    return int(a.shape[0]), r.astype(np.int64), c.astype(np.int64), a[r, c], a.shape


def _entries(M):
    """(shape, layout, rows, cols, values) of a square matrix: host index
    arrays as pxs_lower_union takes them and the values (a numpy array, or a
    torch tensor on M's device) they point into.  A position may occur twice;
    _as_coo sums such entries."""
    import scipy.sparse as sp
    try:
        import torch
    except ImportError:          # pragma: no cover
        torch = None
    if torch is not None and isinstance(M, torch.Tensor):
        if M.layout == torch.sparse_csr:
            return tuple(M.shape), 1, M.crow_indices().cpu().numpy(), M.col_indices().cpu().numpy(), M.values()
        if M.layout == torch.sparse_csc:
            return tuple(M.shape), 2, M.row_indices().cpu().numpy(), M.ccol_indices().cpu().numpy(), M.values()
        if M.layout == torch.sparse_coo:
            M = M.coalesce()
            idx = M.indices().cpu().numpy()
            return tuple(M.shape), 0, idx[0], idx[1], M.values()
    elif sp.issparse(M) and M.format in ("csr", "csc"):
        if M.format == "csr":
            return tuple(M.shape), 1, M.indptr, M.indices, M.data
        return tuple(M.shape), 2, M.indices, M.indptr, M.data
    n, r, c, v, shape = _as_coo(M)
    return tuple(shape), 0, r, c, v


def _union(H, S):
    """(n, colptr, rowind, (hsrc, values of H), (ssrc, values of S)): the
    pattern of lower_csc with the sources of its values (binding.lower_union)."""
    h, s = _entries(H), _entries(S)
    for again in (False, True):
        if len(h[0]) != 2 or h[0][0] != h[0][1] or h[0] != s[0]:
            raise ValueError(f"H and S must be square of one size, got {h[0]} and {s[0]}")
        n = int(h[0][0])
        colptr, rowind, hsrc, ssrc, dup = B.lower_union(n, h[1:4], s[1:4])
        if not dup or again:
            break
        h, s = ((x[4], 0, x[1], x[2], x[3]) for x in (_as_coo(H), _as_coo(S)))   # sums the entries of one position
    return n, colptr, rowind, (hsrc, h[4]), (ssrc, s[4])


def _take(src, vals, dt):
    """The values at their sources: zero where there is none (-1), conjugated
    where the entry is mirrored (-2 - index) and complex."""
    if not isinstance(vals, np.ndarray):
        vals = vals.cpu().numpy()
    out = np.zeros(src.shape[0], dtype=dt)
    low, mir = src >= 0, src < -1
    if low.all():
        out[:] = vals[src]
        return out
    out[low] = vals[src[low]]
    out[mir] = vals[-2 - src[mir]]
    if np.iscomplexobj(out):
        out[mir] = np.conj(out[mir])
    return out


def lower_csc(H, S):
    """(n, colptr int64, rowind int32, hval, sval): the lower triangle of
    pattern(H) U pattern(S) in CSC (rows sorted, diagonal included), values
    aligned with it (zero where a matrix has no entry).  Lower entries win;
    an entry present only above the diagonal is mirrored, conjugated when the
    values are complex."""
    n, colptr, rowind, h, s = _union(H, S)
    dt = np.complex128 if _is_complex(h[1]) or _is_complex(s[1]) else np.float64
    return n, colptr, rowind, _take(*h, dt), _take(*s, dt)


def _is_complex(v):
    return np.iscomplexobj(v) if isinstance(v, np.ndarray) else v.is_complex()


_NUMPY_TYPES = {"torch." + t for t in ("float64", "float32", "float16", "complex128", "complex64", "int64", "int32",
                                       "int16", "int8", "uint8", "bool")}


def _index_arrays(M):
    """The index tensors of a torch sparse matrix on the device (coalesced
    coordinates, compressed rows or columns) and its values; None for any
    other input, and for values that the host path refuses or may refuse (with
    gradients, lazily conjugated, or of a type numpy does not have), so that
    they are refused whether or not their pattern has been seen."""
    try:
        import torch
    except ImportError:          # pragma: no cover
        return None
    if not isinstance(M, torch.Tensor) or not M.is_cuda:
        return None
    if M.layout == torch.sparse_csr:
        out = M.crow_indices(), M.col_indices(), M.values()
    elif M.layout == torch.sparse_csc:
        out = M.ccol_indices(), M.row_indices(), M.values()
    elif M.layout == torch.sparse_coo:
        M = M.coalesce()
        out = M.indices(), M.values()
    else:
        return None
    v = out[-1]
    if v.requires_grad or v.is_conj() or v.is_neg() or v.dim() != 1 or str(v.dtype) not in _NUMPY_TYPES:
        return None
    return out


# What a solver keeps of the patterns it has seen on the device: the value maps of
# the MAPS_KEPT most recently used ones and at most MAPS_BYTES of device memory
# (one map where that alone is larger).  A map takes 24 to 50 bytes per entry of
# H (0.2 GB for a sheet of N = 26,624 in compressed rows).
MAPS_KEPT = 16
MAPS_BYTES = 1 << 30


class _ValueMap:
    """The device-side part of lower_csc for one pair of input patterns:
    copies of their index arrays, compared in full with those of a later
    input, and for every stored entry the source of its value."""

    def __init__(self, key, index, h, s, device):
        import torch
        self.key = key
        self.index = [t.clone() for t in index]
        self.maps = []
        for src, _ in (h, s):
            low = torch.from_numpy(np.where(src >= 0, src, np.where(src < -1, -2 - src, 0))).to(device)
            none = torch.from_numpy(src == -1).to(device) if np.any(src == -1) else None
            mir = torch.from_numpy(src < -1).to(device) if np.any(src < -1) else None
            self.maps.append((low, none, mir))
        held = [*self.index, *(t for m in self.maps for t in m if t is not None)]
        self.bytes = sum(t.numel() * t.element_size() for t in held)
        # complete before another stream or thread can find it
        torch.cuda.current_stream(device).synchronize()

    def matches(self, key, index):
        import torch
        return key == self.key and all(a.shape == b.shape and torch.equal(a, b) for a, b in zip(self.index, index))

    def values(self, which, vals, cplx):
        import torch
        low, none, mir = self.maps[which]
        dt = torch.complex128 if cplx else torch.float64
        if vals.numel() == 0:
            return torch.zeros(low.shape[0], dtype=dt, device=low.device)
        out = vals.to(dt).index_select(0, low)
        if mir is not None and cplx:
            out = torch.where(mir, out.conj(), out)
        if none is not None:
            out = out.masked_fill(none, 0.0)
        return out


def spectrum_bound(colptr, rowind, hval, sval):
    """A bound on max |eps| over the pencil's eigenvalues, from Gershgorin:
    ||H||_2 <= max_i sum_j |H_ij| and lambda_min(S) >= min_i (S_ii - sum_{j != i} |S_ij|).
    None when S is not strictly diagonally dominant."""
    n = colptr.shape[0] - 1
    cols = np.repeat(np.arange(n), np.diff(colptr))
    rows = rowind.astype(np.int64)
    off = rows != cols
    ah, as_ = np.abs(hval), np.abs(sval)
    hrow = np.bincount(rows, ah, minlength=n) + np.bincount(cols[off], ah[off], minlength=n)
    srow = np.bincount(rows[off], as_[off], minlength=n) + np.bincount(cols[off], as_[off], minlength=n)
    sdiag = np.zeros(n)
    sdiag[rows[~off]] = np.real(sval[~off])
    lo = float(np.min(sdiag - srow))
    if lo <= 0.0:
        return None
    return float(np.max(hrow)) / lo


def pencil_dE(colptr, rowind, hval, sval, mu):
    """Delta E of the pole table for a pencil given on its lower triangle:
    the Gershgorin bound on max |eps| plus |mu|, which bounds max |eps - mu|
    over the spectrum.  Raises ValueError when S is not strictly diagonally
    dominant (then the caller must give Delta E)."""
    bound = spectrum_bound(colptr, rowind, hval, sval)
    if bound is None:
        raise ValueError("S is not strictly diagonally dominant: pass dE, a bound on max |eps - mu|")
    return bound + abs(mu)


def _on(stream):
    """Makes stream torch's current stream for the block (None: unchanged),
    so uploads, allocations and the library's launches share one stream."""
    if stream is None:
        return contextlib.nullcontext()
    import torch
    return torch.cuda.stream(stream)


class Solver:
    """Keeps one symbolic analysis per sparsity pattern (bound to the
    device) and the last factor/workspace buffers of each; analysis options
    (leaf_cols, panel_width, ...) apply to every pattern."""

    def __init__(self, device="cuda", **analysis_options):
        self.device = device
        self.options = analysis_options
        self._cache = {}
        self._maps = []              # (cache entry, value map), most recently used first
        self._lock = threading.Lock()

    def _entry(self, n, colptr, rowind, blocks, coords):
        h = hashlib.sha1()
        h.update(np.int64(n).tobytes())
        h.update(colptr.tobytes())
        h.update(rowind.tobytes())
        key = h.hexdigest()
        e = self._cache.get(key)
        if e is None:
            a = B.Analysis(n, colptr, rowind, blkptr=blocks, coords=coords, **self.options)
            a.bind(self.device)
            import torch
            e = {"analysis": a, "buffers": {},
                 "colptr": torch.from_numpy(colptr).to(self.device),
                 "rowind": torch.from_numpy(rowind.astype(np.int64)).to(self.device),
                 "colptr_host": colptr, "rowind_host": rowind, "maps": []}
            self._cache[key] = e
        return e

    def _keep(self, e, m):
        """Makes m the most recently used map and drops those over the bounds:
        more than two of one entry, MAPS_KEPT or MAPS_BYTES in all."""
        with self._lock:
            if self._maps and self._maps[0][1] is m:
                return
            kept, here, held = [], 0, 0
            for q, x in [(e, m)] + [(q, x) for q, x in self._maps if x is not m]:
                here += q is e
                held += x.bytes
                if not kept or (len(kept) < MAPS_KEPT and held <= MAPS_BYTES and not (q is e and here > 2)):
                    kept.append((q, x))
                else:
                    held -= x.bytes
            self._maps = kept
            for q in list(self._cache.values()):
                q["maps"] = [x for r, x in kept if r is q]

    def _pencil(self, H, S, blocks, coords):
        """(cache entry, H values, S values on the device, value map or None).
        Sparse tensors on the device whose index arrays equal those of an
        earlier call (compared in full there, the latest first) have their
        values gathered on the device; everything else goes through the host.
        The caller holds the map until its work on the values is done: another
        thread may drop it here."""
        import torch
        hi, si = _index_arrays(H), _index_arrays(S)
        index = key = None
        if hi is not None and si is not None and H.shape == S.shape and H.device == S.device:
            index = [*hi[:-1], *si[:-1]]
            key = (H.layout, S.layout, tuple(H.shape), H.device, *(t.dtype for t in index))
            cplx = hi[-1].is_complex() or si[-1].is_complex()
            for e, m in list(self._maps):
                if m.matches(key, index):
                    self._keep(e, m)
                    return e, m.values(0, hi[-1], cplx), m.values(1, si[-1], cplx), m
        n, colptr, rowind, h, s = _union(H, S)
        dt = np.complex128 if _is_complex(h[1]) or _is_complex(s[1]) else np.float64
        e = self._entry(n, colptr, rowind, blocks, coords)
        Hd, Sd = (torch.from_numpy(_take(*x, dt)).to(self.device) for x in (h, s))
        # (entries summed into one position have other values than the input's)
        if index is not None and Hd.device == H.device and h[1].shape == hi[-1].shape and s[1].shape == si[-1].shape:
            self._keep(e, _ValueMap(key, index, h, s, Hd.device))
        return e, Hd, Sd, None

    def _buffers(self, e, kind, P):
        import torch
        a = e["analysis"]
        b = e["buffers"].get(kind)
        if b is None or b[0] != P:
            e["buffers"].pop(kind, None)
            if kind == "herm":
                lb, wb = B.hermitian_sizes(a, P)
                L = torch.empty(lb, dtype=torch.uint8, device=self.device)
                W = torch.empty(wb, dtype=torch.uint8, device=self.device)
            else:
                L, W = a.buffers(P, device=self.device)
            b = (P, L, W)
            e["buffers"][kind] = b
        return b[1], b[2]

    def check_overlap(self, H, S, blocks=None, coords=None, stream=None):
        """Whether S is positive definite, as the pencil needs (Sec. II.A),
        checked on the device on the pattern of (H, S): real S by the
        inertia of S (Sylvester: the number of negative pivots of its
        L D L^T), complex Hermitian S by the pivots of its L D U, which are
        real and all positive exactly when S is.  Returns (ok, number of
        non-positive pivots, tiny-pivot column or 0)."""
        n, colptr, rowind, hval, sval = lower_csc(H, S)
        with _on(stream):
            import torch
            e = self._entry(n, colptr, rowind, blocks, coords)
            a = e["analysis"]
            Sd = torch.from_numpy(sval).to(self.device)
            Z = torch.zeros_like(Sd)
            if np.iscomplexobj(sval):
                f = B.HermitianFactorization(a, Sd, Z, np.array([0j]))
                info = int(f.info[0])
                d = f.diag(0).cpu().numpy()
                bad = int(np.sum(d.real <= 0.0))
            else:
                neg, inf = B.inertia(a, Sd, Z, np.array([0.0]))
                info, bad = int(inf[0]), int(neg[0])
        return info == 0 and bad == 0, bad, info

    def density_matrix(self, H, S, mu, beta, P, outputs=("rho", "E"), dE=None, blocks=None, coords=None,
                       stream=None, check_overlap=False):
        """Returns (*matrices in the order of `outputs`, traces dict).  Each
        matrix is a torch sparse CSC tensor of the lower triangle of the
        union pattern on the device (float64, complex128 for Hermitian
        input).  traces: N = Tr(G S), Eband = Tr(G H), and with the sets
        asked for TrES = Tr(G^E S), free_energy = Tr(G^F S) + mu N,
        dN_dmu = Tr(G^d S); info = per-shift tiny-pivot columns (0 = none).
        check_overlap runs check_overlap first and raises ValueError when S
        is not positive definite.  stream: a torch.cuda.Stream for every
        upload, allocation and launch of the call (default: the current
        stream)."""
        with _on(stream):
            return self._density_matrix(H, S, mu, beta, P, outputs, dE, blocks, coords, check_overlap)

    def _density_matrix(self, H, S, mu, beta, P, outputs, dE, blocks, coords, check_overlap):
        import torch
        outputs = tuple(outputs)
        if not outputs or any(o not in SETS for o in outputs):
            raise ValueError(f"outputs must be a non-empty subset of {SETS}")
        if check_overlap:
            ok, bad, info = self.check_overlap(H, S, blocks=blocks, coords=coords)
            if not ok:
                raise ValueError(f"S is not positive definite: {bad} non-positive pivots, tiny pivot at {info}")
        nsets = 1 + max(SETS.index(o) for o in outputs)
        e, Hd, Sd, held = self._pencil(H, S, blocks, coords)   # held: see _pencil
        a = e["analysis"]
        n = a.n
        herm = Hd.is_complex()
        if dE is None:
            dE = pencil_dE(e["colptr_host"], e["rowind_host"], Hd.cpu().numpy(), Sd.cpu().numpy(), mu)
        if herm:
            L, W = self._buffers(e, "herm", P)
            sh, wt = B.poles(beta, dE, mu, P, nsets)
            f = B.HermitianFactorization(a, Hd, Sd, sh, L=L, work=W)
            info = f.info.copy()
            f.selinv()
            out, tr = f.pole_sum(wt)
            del f
        else:
            L, W = self._buffers(e, "real", P)
            out, tr, info, sh, wt = B.density_matrix(a, Hd, Sd, beta, dE, mu, P, nsets=nsets, L=L, work=W)
        mats = []
        for o in outputs:
            g = SETS.index(o)
            mats.append(torch.sparse_csc_tensor(e["colptr"], e["rowind"], out[g], size=(n, n)))
        N = float(tr[0, 0])
        traces = {"N": N, "Eband": float(tr[0, 1]), "dE": float(dE), "info": info}
        if nsets > 1:
            traces["TrES"] = float(tr[1, 0])
        if nsets > 2:
            traces["free_energy"] = float(tr[2, 0]) + mu * N
        if nsets > 3:
            traces["dN_dmu"] = float(tr[3, 0])
        return (*mats, traces)


_default = None


def density_matrix(H, S, mu, beta, P, outputs=("rho", "E"), dE=None, blocks=None, coords=None, stream=None,
                   check_overlap=False):
    """Solver.density_matrix on a module-level solver (device cuda)."""
    global _default
    if _default is None:
        _default = Solver()
    return _default.density_matrix(H, S, mu, beta, P, outputs=outputs, dE=dE, blocks=blocks, coords=coords,
                                   stream=stream, check_overlap=check_overlap)
