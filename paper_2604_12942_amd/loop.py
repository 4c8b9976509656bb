"""Gaussian-based loop closure (Sec. III-D): registration of a loopframe's Gaussians against the
map Gaussians seen from the views around a historical loopframe (Eq. 13-16), with the
acceptance test, and propagation of a corrected pose to a segment of the map.

Registration runs on the device end to end (set extraction, covariances, grid, Gauss-Newton with
an on-device 6x6 solve).  The host queues 8 iterations, then as many again as it has queued so far, and
reads the statistics after each batch: iterations after convergence do nothing, but their launches cost
the host up to 18 us each (a registration that converged after 6 of 30: 776 -> 654 us).
"""
from __future__ import annotations

import numpy as np
import torch

from . import gicp_iterate, gicp_prepare

# readings: correspondences within 0.5 m; queries limited to 30 m from a keyframe centre;
# accepted when converged with at least 100 correspondences and mean r^T W r below 1
D_CORR, D_MAX = 0.5, 30.0
MIN_CORR, ACCEPT_COST = 100, 1.0


def _lie_together(state):
    """Whether the statistics, set sizes and pose of a state are parts of its one buffer, as gicp_prepare lays
    them out.  In a copy of a state (cloned, moved or loaded tensor by tensor) they are not."""
    if "buf" not in state or "pose" not in state:
        return False
    at = state["buf"].data_ptr()
    return (state["stats"].data_ptr() == at and state["counts"].data_ptr() == at + 320 and
            state["pose"].data_ptr() == at + 328)


def register(P, sh_degree, segment_id, src_segment, cams, n_cams, pose0=None, d_max=D_MAX, d_corr=D_CORR,
             max_iter=30, state=None):
    """Aligns the Gaussians of segment src_segment to the target set seen from cams (device
    gsr_camera records).  pose0: (R [3, 3], t [3]) initial guess (identity by default).
    Returns a dict with R, t, converged, failed, iterations, count, cost, rmse, accepted, state."""
    dev = P["means"].device
    R0, t0 = (np.eye(3), np.zeros(3)) if pose0 is None else pose0
    start = torch.tensor(np.concatenate([np.asarray(R0, np.float64).ravel(), np.asarray(t0, np.float64)]),
                         dtype=torch.float64, device=dev)
    state = gicp_prepare(P, sh_degree, segment_id, src_segment, cams, n_cams, d_max, d_corr, state)
    together = _lie_together(state)
    pose = start
    if together:
        pose = state["pose"]
        pose.copy_(start)
    queued = 0
    while True:
        batch = min(queued or 8, max_iter - queued)
        gicp_iterate(P, sh_degree, state, pose, batch)
        queued += batch
        if together:
            host = state["buf"].cpu().numpy()
        else:
            host = np.concatenate([state["stats"].cpu().numpy(), state["counts"].cpu().numpy().view(np.float64),
                                   pose.cpu().numpy()])
        if host[36] or host[38] or queued >= max_iter:  # converged, failed
            break
    st, pz, sizes = host[:40], host[41:], host[40:41].view(np.int32)
    count = int(st[29])
    conv, failed = bool(st[36]), bool(st[38])
    cost = float(st[27])
    accepted = conv and not failed and count >= MIN_CORR and cost / count < ACCEPT_COST
    return dict(R=pz[:9].reshape(3, 3), t=pz[9:], converged=conv, failed=failed, iterations=int(st[37]),
                count=count, cost=cost, rmse=float(np.sqrt(st[28] / max(count, 1))), accepted=accepted,
                n_src=int(sizes[0]), n_tgt=int(sizes[1]), state=state)
