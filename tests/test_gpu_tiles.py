"""The mixed-radix line, plane and tile kernels at the sizes where their plans
change, against the FP64 oracle: planes just inside and past LDS, axes of one
to five factors, odd and even last factors, tiles with a ragged edge, and pair
sums shared by several workgroups over several launches.  FP32 paths: relative
L2 error <= 1e-5 (the bound of every FP32 path); 16-bit scores: the storage
bound, and the reconstruction of the dequantised scores to 1e-5 (complex64
intermediates)."""
import hashlib
import json
import os

import numpy as np
import pytest

import oracle as O
from paper_1505_07690_amd import inputs

pytestmark = pytest.mark.gpu

TOL = 1e-5


def rel(a, b):
    a, b = np.asarray(a), np.asarray(b)
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def _random_orients(n, seed):
    v = np.random.default_rng(seed).standard_normal((n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


SHAPES = {
    "plane_19200_of_lds": ((4, 128, 150), "octahedron"),   # 15 x 10 rows, 19 values per thread
    "plane_past_lds": ((5, 180, 150), "octahedron"),       # y lines and x lines, ragged x chunks
    "padded_rows_past_lds": ((3, 160, 128), "octahedron"),  # 20480 values, but padded rows
    "x_one_factor": ((9, 60, 16), "tetrahedron"),
    "y_one_factor": ((16, 12, 225), "tetrahedron"),
    "z_three_factors": ((250, 6, 10), "octahedron"),
    "z_five_factors": ((3125, 2, 4), "octahedron"),
    "y_4050": ((2, 4050, 3), "tetrahedron"),
    "x_4096": ((3, 2, 4096), "octahedron"),
    "three_factor_plane": ((6, 81, 162), "tetrahedron"),
    "sum_shared_over_launches": ((12, 16, 18), 140),       # 140 stored rows: two launches
    "sum_shared_one_launch": ((48, 20, 24), 30),
    # planes past LDS: a factor of y goes with the z lines
    "split_2_ragged_sum_shared": ((5, 162, 150), 30),      # 81 x 150 lines: not a multiple of 32
    "split_4": ((3, 200, 250), "tetrahedron"),
    "split_8_one_factor_z": ((2, 240, 405), "octahedron"),
    "split_2_z_12_rows": ((36, 120, 180), "tetrahedron"),
    "split_past_threads": ((243, 16, 1296), "tetrahedron"),  # z tile too large: three passes
    "split_odd_y": ((3, 225, 100), "octahedron"),            # three passes
}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_tile_plans(name):
    import torch
    from paper_1505_07690_amd import os3d
    shape, kind = SHAPES[name]
    n = _random_orients(kind, 77) if isinstance(kind, int) else inputs.platonic_orientations(kind)
    p = O.WaveletParams(L=5, s_theta=inputs.s_theta_for(len(n)))
    vol = inputs.tubes(shape, 2, 1.2, 0.1, 0, 61)
    ob = O.build_bank(shape, n, p)
    gb = os3d.Bank(shape, n, p)
    f = torch.from_numpy(vol).cuda()
    U, _ = os3d.forward(f, gb)
    Uo = O.forward(vol.astype(np.float64), ob)
    assert rel(U.cpu().numpy(), Uo) < TOL
    rng = np.random.default_rng(5)
    Un = (rng.standard_normal(Uo.shape) + 1j * rng.standard_normal(Uo.shape)).astype(np.complex64)
    Ut = torch.from_numpy(Un).cuda()
    assert rel(os3d.reconstruct(Ut, gb).cpu().numpy(), O.reconstruct(Un.astype(np.complex128), ob)) < TOL
    assert rel(os3d.adjoint(Ut, gb).cpu().numpy(), O.adjoint(Un.astype(np.complex128), ob)) < TOL
    gp = os3d.process(f, gb, "identity").cpu().numpy()
    assert rel(gp, O.reconstruct(Uo, ob)) < TOL
    for fmt, bound in (("bf16", 4e-3), ("fp16", 5e-4)):
        Uq, sc = os3d.forward(f, gb, dtype=fmt)
        Ud = os3d.unpack16(Uq, sc, fmt).cpu().numpy()
        assert rel(Ud, Uo) < bound
        rq = os3d.reconstruct(Uq, gb, scales=sc, dtype=fmt).cpu().numpy()
        assert rel(rq, O.reconstruct(Ud.astype(np.complex128), ob)) < TOL


# Planes past LDS whose y lines begin with a stage of two factors: the 16-bit
# forward transform takes z, y and x lines there.
@pytest.mark.parametrize("shape", [(3, 150, 150), (3, 108, 200), (2, 243, 90), (2, 135, 160), (2, 90, 240)])
def test_16_bit_scores_of_planes_past_lds(shape):
    import torch
    from paper_1505_07690_amd import os3d
    n = inputs.platonic_orientations("octahedron")
    p = O.WaveletParams(L=5, s_theta=inputs.s_theta_for(len(n)))
    vols = [inputs.tubes(shape, 2, 1.2, 0.1, 0, s) for s in (71, 72)]
    gb = os3d.Bank(shape, n, p)
    ob = O.build_bank(shape, n, p)
    f = torch.from_numpy(np.stack(vols)).cuda()
    for fmt, bound in (("bf16", 4e-3), ("fp16", 5e-4)):
        U, sc = os3d.forward(f, gb, dtype=fmt)
        for i, vol in enumerate(vols):
            Ua, sa = os3d.forward(f[i].contiguous(), gb, dtype=fmt)
            assert torch.equal(Ua, U[i]) and torch.equal(sa, sc[i])
            Ud = os3d.unpack16(Ua, sa, fmt).cpu().numpy()
            assert rel(Ud, O.forward(vol.astype(np.float64), ob)) < bound


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_soft_threshold_of_tile_plans(name):
    """A Phi that commutes with no pass of the transform, on every plan."""
    import torch
    from paper_1505_07690_amd import os3d
    shape, kind = SHAPES[name]
    n = _random_orients(kind, 78) if isinstance(kind, int) else inputs.platonic_orientations(kind)
    p = O.WaveletParams(L=5, s_theta=inputs.s_theta_for(len(n)))
    vol = inputs.tubes(shape, 2, 1.2, 0.1, 0, 62)
    ob = O.build_bank(shape, n, p)
    got = os3d.process(torch.from_numpy(vol).cuda(), os3d.Bank(shape, n, p), "soft_threshold", 1.5).cpu().numpy()
    assert rel(got, O.process(vol.astype(np.float64), ob, "soft_threshold", 1.5)) < TOL


@pytest.mark.parametrize("name", ["sum_shared_over_launches", "sum_shared_one_launch", "split_2_ragged_sum_shared",
                                  "split_odd_y", "three_factor_plane"])
def test_batches_of_tile_plans(name):
    """A batch of two equals its volumes run alone (the sums of one volume are reused by the next)."""
    import torch
    from paper_1505_07690_amd import os3d
    shape, kind = SHAPES[name]
    n = _random_orients(kind, 79) if isinstance(kind, int) else inputs.platonic_orientations(kind)
    gb = os3d.Bank(shape, n, O.WaveletParams(L=5, s_theta=inputs.s_theta_for(len(n))))
    f = torch.from_numpy(np.stack([inputs.tubes(shape, 2, 1.2, 0.1, 0, s) for s in (63, 64)])).cuda()
    one = [f[i].contiguous() for i in range(2)]
    gp = os3d.process(f, gb, "soft_threshold", 1.5)
    for i in range(2):
        assert torch.equal(gp[i], os3d.process(one[i], gb, "soft_threshold", 1.5))
    for fmt in ("c64", "bf16"):
        U, sc = os3d.forward(f, gb, dtype=fmt)
        r = os3d.reconstruct(U, gb, scales=sc, dtype=fmt)
        for i in range(2):
            Ua, sa = os3d.forward(one[i], gb, dtype=fmt)
            assert torch.equal(Ua, U[i]) and (sc is None or torch.equal(sa, sc[i]))
            assert torch.equal(os3d.reconstruct(Ua, gb, scales=sa, dtype=fmt), r[i])


# Stored 16-bit scores are the same words from one version of the library to
# the next (they are files and baselines of its users): SHA-256 prefixes of the
# words and scales, bf16 and fp16, from the library before its line and tile
# kernels.  One grid per route and per kind of butterfly.
with open(os.path.join(os.path.dirname(__file__), "golden", "score_words.json")) as _f:
    WORDS = json.load(_f)


@pytest.mark.parametrize("name", sorted(WORDS))
def test_stored_words(name):
    import torch
    from paper_1505_07690_amd import os3d
    shape = tuple(int(x) for x in name.split("x"))
    n = inputs.platonic_orientations("octahedron") if np.prod(shape) > 2e5 else inputs.icosahedral_orientations(0)
    gb = os3d.Bank(shape, n, os3d.make_params(L=5, s_theta=inputs.s_theta_for(len(n))))
    f = torch.from_numpy(inputs.tubes(shape, 3, 1.3, 0.1, 0, 90)).cuda()
    got = []
    for fmt in ("bf16", "fp16"):
        U, sc = os3d.forward(f, gb, dtype=fmt)
        got.append(hashlib.sha256(U.cpu().numpy().tobytes() + sc.cpu().numpy().tobytes()).hexdigest()[:16])
    assert got == WORDS[name]
