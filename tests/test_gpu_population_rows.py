"""Row copies of the population steps at the sizes where they can go wrong
(block boundaries, every SH width, arrays off the 16-byte alignment, with
and without moments) vs the oracle, on the GPU.  Copied rows are exact;
computed centres and distances carry one float32 rounding of a double
result (2^-24 relative, 1e-6 with the centre's cancellation)."""
import numpy as np
import pytest
import torch

from oracle import population as POP
from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd.population import PopulationControl

pytestmark = pytest.mark.gpu
FIELDS = ("means", "quats", "dists", "opacity", "sh")


def _state(kind, n, degree, seed):
    rng = np.random.default_rng(seed)
    nd = 3 if kind == L.OCTAHEDRON else 4
    K = (degree + 1) ** 2
    params = {"means": rng.normal(size=(n, 3)), "quats": rng.normal(size=(n, 4)),
              "dists": np.exp(rng.uniform(np.log(0.01), np.log(3.0), size=(n, nd))),
              "opacity": rng.uniform(0.0, 0.2, size=n), "sh": rng.normal(size=(n, K, 3))}
    params = {k: v.astype(np.float32) for k, v in params.items()}
    moments = {(w, k): rng.normal(size=params[k].shape).astype(np.float32) for w in ("m", "v") for k in params}
    stats = {"grad_accum": rng.uniform(0, 1.2e-3, size=n).astype(np.float32),
             "count": rng.integers(0, 5, size=n).astype(np.int32),
             "max_radius": rng.uniform(0, 40, size=n).astype(np.float32)}
    return params, moments, stats, rng.normal(size=(n, 2, 3)).astype(np.float32)


def _dev(a, shift):
    """A device copy that starts `shift` floats into its allocation."""
    a = np.ascontiguousarray(a)
    buf = torch.empty(a.size + shift, dtype=torch.float32, device="cuda")
    buf[shift:] = torch.as_tensor(a, device="cuda").reshape(-1)
    return buf[shift:].view(a.shape)


@pytest.mark.parametrize("kind", [L.OCTAHEDRON, L.TETRAHEDRON])
@pytest.mark.parametrize("n,degree,shift,with_moments", [(1023, 0, 0, True), (1024, 1, 0, True), (1025, 2, 1, True),
                                                         (2049, 3, 3, True), (3000, 3, 0, False), (2, 1, 2, False)])
def test_densify_rows(kind, n, degree, shift, with_moments):
    print(f"densify rows kind={kind} n={n} degree={degree} shift={shift}", flush=True)
    params, moments, stats, normals = _state(kind, n, degree, seed=n + degree)
    P = {k: _dev(params[k], shift) for k in FIELDS}
    M = {k: _dev(moments[("m", k)], shift) for k in FIELDS} if with_moments else None
    V = {k: _dev(moments[("v", k)], shift) for k in FIELDS} if with_moments else None
    pc = PopulationControl(kind, degree, n)
    pc.grad_accum.copy_(torch.as_tensor(stats["grad_accum"]))
    pc.count.copy_(torch.as_tensor(stats["count"]))
    pc.max_radius.copy_(torch.as_tensor(stats["max_radius"]))
    newp, newm, newv = pc.densify(P, 10.0, M, V, normals=torch.as_tensor(normals, device="cuda"))
    ref_p, ref_m = POP.densify(kind, params, moments, stats, 10.0, normals)
    assert newp["means"].shape[0] == ref_p["means"].shape[0]
    for k in ("quats", "opacity", "sh"):
        assert np.array_equal(newp[k].cpu().numpy().astype(np.float64), ref_p[k]), k
    for k in ("means", "dists"):
        np.testing.assert_allclose(newp[k].cpu().numpy(), ref_p[k], rtol=1e-6, atol=1e-6, err_msg=k)
    if not with_moments:
        assert newm is None and newv is None
        return
    for k in FIELDS:
        assert np.array_equal(newm[k].cpu().numpy().astype(np.float64), ref_m[("m", k)]), k
        assert np.array_equal(newv[k].cpu().numpy().astype(np.float64), ref_m[("v", k)]), k
