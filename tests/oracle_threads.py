"""The oracle's array steps in threads (test infrastructure).

Full-size GPU tests spend most of their time in the oracle's phasors and transforms, one thread of
numpy.  Channels are independent in both, and bins are independent in the sum over channels, so the
steps run in slices of those, each by the oracle's own function: the results are the same, bit for
bit.  Small arrays go to the oracle directly.
"""
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np

SMALL = 1 << 20                     # elements
WORKERS = min(16, os.cpu_count() or 1)


def _slices(n: int):
    step = -(-n // WORKERS)
    return [slice(a, min(n, a + step)) for a in range(0, n, step)]


def install(module, small: int = SMALL):
    """Replace the module's steps; returns the function that puts them back."""
    own = module.phasors, module.forward_spectra, module.phasor_sum
    pool = ThreadPoolExecutor(WORKERS)

    def split(n, shape, dtype, call, at):
        out = np.empty(shape, dtype=dtype)

        def one(s):
            out[at(s)] = call(s)
        list(pool.map(one, _slices(n)))
        return out

    def phasors(tau_row, L, mode):
        tau = np.asarray(tau_row)
        if tau.size * (L // 2 + 1) < small:
            return own[0](tau_row, L, mode)
        return split(tau.size, (tau.size, L // 2 + 1), np.complex128, lambda s: own[0](tau[s], L, mode), lambda s: s)

    def forward_spectra(seg):
        if seg.ndim != 2 or seg.size < small:
            return own[1](seg)
        return split(seg.shape[0], (seg.shape[0], seg.shape[1] // 2 + 1), np.complex128, lambda s: own[1](seg[s]), lambda s: s)

    def phasor_sum(W, X):
        if W.ndim != 2 or W.shape != X.shape or W.size < small:
            return own[2](W, X)
        return split(W.shape[1], W.shape[1], np.complex128, lambda s: own[2](W[:, s], X[:, s]), lambda s: s)

    module.phasors, module.forward_spectra, module.phasor_sum = phasors, forward_spectra, phasor_sum

    def undo():
        module.phasors, module.forward_spectra, module.phasor_sum = own
        pool.shutdown()
    return undo
