"""Helpers for the GPU parity tests: move numpy arrays to the device, run the HIP path
through the C ABI binding, bring results back as numpy."""
import numpy as np
import torch


def dev(a):
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    a = t.detach().cpu().numpy()
    return a


def host_u32(t):
    return host(t).view(np.uint32)


def gemm_tolerance_ok(orc, y_gpu, y_ref, t_ref):
    """|y_gpu - y_ref| <= 1e-3 * sum_k |x w_hat| + 1 fp16 ulp, per element."""
    err = np.abs(y_gpu.astype(np.float64) - y_ref)
    tol = 1e-3 * t_ref + orc.ulp16(y_ref)
    bad = err > tol
    return not bad.any(), float((err / tol).max()), int(bad.sum())


def silu_tolerance(orc, y_ref, t_ref):
    """Bound on |h_gpu - h_ref| for h = SiLU(g) u from the GEMM bound |dg| <= 1e-3 t_g,
    |du| <= 1e-3 t_u on the fp32 sums: |dh| <= |SiLU'(g)| |u| |dg| + |SiLU(g)| |du| + |dg||du|,
    |SiLU'| <= 1.1; plus the hardware exponential (1e-6 relative) and the final fp16 rounding."""
    g, u = y_ref[:, 0::2], y_ref[:, 1::2]
    dg, du = 1e-3 * t_ref[:, 0::2], 1e-3 * t_ref[:, 1::2]
    h = orc.silu_mul_ref(g, u)
    return h, 1.1 * np.abs(u) * dg + np.abs(orc.silu_ref(g)) * du + 1.1 * dg * du + 1e-6 * np.abs(h) + orc.ulp16(h)
