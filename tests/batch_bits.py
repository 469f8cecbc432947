"""Droplet sweeps whose fields are held to the bit (test_gpu_batch_bits.py).

The initial densities are rational functions of the node's integers, so that
every machine starts from the same doubles."""
import zlib

import numpy as np

STEPS = 301   # three checks, and a step that a two-step launch leaves over
EVERY = 100
# (side, order, G, tau, initialisation); the first four blow up, and are retired
# with a field that is finite on a part of the nodes
ITEMS = [(75, 4, -5.30, 0.8, "rest"), (88, 4, -5.34, 0.8, "rest"), (88, 4, -5.34, 0.8, "equilibrium"),
         (100, 4, -5.34, 0.8, "rest"), (64, 4, -5.0, 1.0, "equilibrium"), (97, 6, -5.2, 0.8, "rest"),
         (71, 8, -4.9, 1.2, "equilibrium"), (130, 10, -5.1, 1.0, "rest")]


def density(side):
    """A droplet of radius side / 4 with a +-1e-3 jitter."""
    d = np.arange(side, dtype=np.float64) - side // 2
    q = (d[:, None] * d[:, None] + d[None, :] * d[None, :]) * 16.0 / float(side * side)
    q = q * q
    q = q * q
    q = q * q                       # (r / R)^16
    k = np.arange(side * side, dtype=np.uint64) * np.uint64(2654435761) % np.uint64(1 << 32)
    jitter = (k.astype(np.float64) / 2.0 ** 31 - 1.0).reshape(side, side) * 1e-3
    return 0.15 + 1.85 / (1.0 + q) + jitter


def sweep(Batch, precision, shape, items=ITEMS):
    """[steps, rule, non-finite nodes, CRC-32 of the density's bytes] per item."""
    bt = Batch([dict(rho0=density(s), order=o, G=g, tau=t, init=i, precision=precision) for s, o, g, t, i in items],
               obs_every=EVERY, variant=shape)
    bt.step(STEPS, tol=1e-14)
    out = []
    for k in range(len(items)):
        rho = np.ascontiguousarray(bt.observe(k)["rho"])
        steps, by = bt.status(k)
        bad = ~np.isfinite(rho)
        rho[bad] = 0.0              # a NaN's payload is not held to anything
        out.append([int(steps), int(by), int(bad.sum()), zlib.crc32(bad.tobytes() + rho.tobytes())])
    bt.close()
    return out
