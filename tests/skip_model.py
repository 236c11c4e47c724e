"""What the posterior kernels skip, in float64: the tests of one tile of 32
low-pass pixels, with sums that have no range to leave.

A tile is tested as a whole: the box of its observations along the principal
axes of the nodes' differences against the boxes of the super-tiles and of the
4 x 4-node chunks.  A pass keeps the chunks bounded less than `depth` (log2)
below the lowest reference (a pixel's best probe, one node per 8 x 8 patch);
the bounds of those left out add up to the skipped weight, which each pixel's
kept weight has to certify; otherwise the next pass goes 4 units deeper, down
to the a-priori threshold.
"""
from __future__ import annotations

from typing import List, NamedTuple, Tuple

import numpy as np

from paper_1706_07263_amd import synth


def scaled_attenuation(hb, hbo2, sigma: float, mu_ref) -> np.ndarray:
    """Scaled log-attenuation of concentrations about mu_ref, [..., 3]."""
    sp = synth.spectra()
    resp = sp.response / sp.response.sum(axis=1, keepdims=True)
    att = np.exp(-sp.path_length_cm * (np.multiply.outer(hb, sp.eps_hb) + np.multiply.outer(hbo2, sp.eps_hbo2)))
    return np.sqrt(np.log2(np.e) / (2.0 * sigma ** 2)) * (-np.log(att @ resp.T) - mu_ref)


class Passes(NamedTuple):
    kept: List[int]        # chunks kept up to and including each pass
    skipped: List[float]   # log2 of the skipped weight after each pass (relative to the lowest reference)
    allowed: List[float]   # log2 of the largest one that every pixel certifies
    moved: float           # largest change of a posterior mean (uM) by what the last pass leaves out


class SkipModel:
    def __init__(self, settings, mu_ref, skip_log2: float, skip_bound: float):
        """settings as synth.plan_settings; mu_ref, skip_log2 and skip_bound
        as the plan reports them (one split)."""
        gt, gs = int(settings["grid_thb"]), int(settings["grid_so2"])
        self.sigma, self.mu_ref = float(settings["sigma"]), np.asarray(mu_ref)
        thb = np.linspace(settings["thb_min"], settings["thb_max"], gt)[:, None]
        so2 = np.linspace(settings["so2_min"], settings["so2_max"], gs)[None, :]
        self.conc = np.stack([thb * (1.0 - so2), thb * so2])                      # [2][gt][gs]
        v = scaled_attenuation(self.conc[0], self.conc[1], self.sigma, self.mu_ref)   # [gt][gs][3]
        side = max(4, min(32, 4 * (min(gt, gs) // 32)))
        assert gt % side == 0 and gs % side == 0, "whole super-tiles"
        sup = v.reshape(gt // side, side, gs // side, side, 3).transpose(0, 2, 1, 3, 4).reshape(-1, side, side, 3)
        chunk = sup.reshape(-1, side // 4, 4, side // 4, 4, 3).transpose(0, 1, 3, 2, 4, 5)   # [sup][ca][cs][4][4][3]
        # principal axes, the strongest last
        few = chunk[::(len(sup) + 63) // 64]
        d = np.concatenate([(few[..., 0, 3, :] - few[..., 0, 0, :]).reshape(-1, 3),
                            (few[..., 3, 0, :] - few[..., 0, 0, :]).reshape(-1, 3)])
        self.axes = np.linalg.eigh(d.T @ d)[1].T                                  # rows
        rot = chunk.reshape(len(sup), -1, 16, 3) @ self.axes.T                    # [sup][chunk][node][axis]
        self.lo, self.hi = rot.min(axis=2), rot.max(axis=2)                       # [sup][chunk][axis]
        patch = min(8, side)
        mid = (patch - 1) // 2
        self.probes = sup[:, mid::patch, mid::patch].reshape(-1, 3) if side % patch == 0 else np.concatenate(
            [sup[:, a + (min(8, side - a) - 1) // 2, b + (min(8, side - b) - 1) // 2]
             for a in range(0, side, 8) for b in range(0, side, 8)])
        self.nodes = chunk.reshape(len(sup), -1, 16, 3)
        order = self.conc.reshape(2, gt // side, side // 4, 4, gs // side, side // 4, 4)
        self.moments = order.transpose(0, 1, 4, 2, 5, 3, 6).reshape(2, len(sup), -1, 16)
        self.skip_log2 = skip_log2
        self.depth0, self.cert = skip_log2, None
        if skip_bound > 0:
            ratio = skip_bound / float(settings["thb_max"])
            self.depth0 = min(skip_log2, max(16.0, -np.log2(0.5 * ratio)))
            self.cert = np.log2(ratio * (1.0 - 1.0 / 16))

    def tiles(self, z: np.ndarray) -> List[np.ndarray]:
        """The tiles of one whole region (128 observations, scaled): 32
        consecutive ones by their coordinate along the strongest axis."""
        assert z.shape == (128, 3)
        return list(z[np.argsort(z @ self.axes[2], kind="stable")].reshape(4, 32, 3))

    def passes(self, z: np.ndarray) -> Passes:
        """All passes of the tile z [32][3]."""
        q = z @ self.axes.T
        far2 = float((np.abs(q).max(axis=0) ** 2).sum())
        slack = 1e-3 + np.sqrt(far2) * 2.0 ** -20
        zlo, zhi = q.min(axis=0) - slack, q.max(axis=0) + slack
        best = -np.min(((z[:, None] - self.probes[None]) ** 2).sum(axis=-1), axis=1)   # [32]
        mmin = best.min() - far2 * 2.0 ** -20

        def bound(lo, hi):
            return -(np.maximum(np.maximum(lo - zhi, zlo - hi), 0.0) ** 2).sum(axis=-1) - mmin

        sv, v = bound(self.lo.min(axis=1), self.hi.max(axis=1)), bound(self.lo, self.hi)
        w = np.exp2(-((z[:, None, None, None] - self.nodes[None]) ** 2).sum(axis=-1) - best[:, None, None, None])
        kept, skipped, allowed = [], [], []
        depth = self.depth0
        while True:
            last = depth >= self.skip_log2
            sup = sv > max(-self.skip_log2, -depth - 12.0)
            keep = sup[:, None] & (v > -depth)
            kept.append(int(keep.sum()))
            mass = 16.0 * (np.exp2(v[sup][~keep[sup]]).sum() + v.shape[1] * np.exp2(sv[~sup]).sum())
            sums = (w * keep[None, :, :, None]).sum(axis=(1, 2, 3))
            skipped.append(float(np.log2(max(mass, 2.0 ** -300))))
            allowed.append(float("inf") if last else float(self.cert + (best + np.log2(sums) - mmin).min()))
            if last or skipped[-1] <= allowed[-1]:
                break
            depth = min(self.skip_log2, depth + 4.0)
        mean = [(self.moments[:, None] * x[None]).sum(axis=(2, 3, 4)) / x.sum(axis=(1, 2, 3))
                for x in (w, w * keep[None, :, :, None])]
        return Passes(kept, skipped, allowed, float(np.abs(mean[0] - mean[1]).max()))


def skip_rule(settings) -> Tuple[float, float]:
    """skip_log2 and skip_bound of a plan of one split with a tolerance > 0."""
    G = int(settings["grid_thb"]) * int(settings["grid_so2"])
    thb_max, tol = float(settings["thb_max"]), float(settings["posterior_tolerance"])
    T = min(160.0, max(16.0, np.ceil(np.log2(2.0 * G * thb_max / tol))))
    if T + 1 >= 160.0:
        return T, (2.0 * G * 2.0 ** -T * thb_max if T < 160.0 else 0.0)
    T += 1
    hard, per_chunk = 2.0 * G * 2.0 ** -T * thb_max, 32.0 * 2.0 ** (6.0 - T) * thb_max
    return T, hard + per_chunk * max(0.0, min(np.floor((tol - hard) / per_chunk), 1e6))
