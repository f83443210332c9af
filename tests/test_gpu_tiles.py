"""Stencil tiles chosen by the size of a launch (small launches cut the z range
and take one vector per tile): the shape never changes a point's arithmetic,
so filtered blocks are bit-identical to whole-box tiles, and the residual's
partial sums differ by their order only."""
import numpy as np
import pytest

from paper_2609_13115_amd import workloads, xls

pytestmark = pytest.mark.gpu


def box(shape, ns, periodic):
    if periodic:
        return workloads.periodic_si_cell(shape[0], ns, workloads.workload_key(1), True)
    return workloads.small_dirichlet(shape[0], ns, shape=shape, h=0.6)


# one column, odd extents, a z range shorter than a chunk, more columns than
# fill the chip with whole boxes, rows wider than a wavefront
@pytest.mark.parametrize("shape,ns,periodic", [((8, 8, 8), 1, True), ((24, 24, 24), 20, True), ((5, 7, 3), 3, False),
                                               ((17, 21, 14), 31, False), ((70, 9, 11), 5, False),
                                               ((20, 33, 45), 150, False), ((13, 12, 1), 2, False),
                                               ((16, 64, 57), 400, False)])
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP64, xls.XLS_PREC_FP32])
def test_chosen_tiles_match_whole_box_tiles(shape, ns, periodic, prec):
    print(f"[case] tiles {shape} ns={ns} periodic={periodic} prec={prec}", flush=True)
    sd = box(shape, ns, periodic)
    lam = np.linspace(-0.2, 0.5, ns)
    out = []
    for whole in (False, True):
        with xls.Subdomain(sd, filter_prec=prec) as s:
            if whole:
                s.xls_subdomain_tune(xls.XLS_PREC_FP64, 0, 0, 0, 1)
                s.xls_subdomain_tune(xls.XLS_PREC_FP32, 0, 0, 0, 1)
            s.xls_subdomain_filter(4, -3.0, 4.0, 45.0)
            out.append((s.xls_subdomain_get_block(), s.xls_subdomain_residual(lam)))
    assert np.array_equal(out[0][0], out[1][0])
    # N_d squares summed in another order: about N_d eps of the sum, twice
    assert np.allclose(out[0][1], out[1][1], rtol=2 * sd.nd * 2.3e-16 + 1e-15, atol=0)


# rows of a pair split by a tile's or the box's edge, tiles whose row pairs do
# not fill the workgroup (row counts trimmed), halo counts on both sides of
# three cells a lane
@pytest.mark.parametrize("shape,ns,periodic", [((46, 23, 7), 3, False), ((24, 24, 24), 5, True), ((33, 37, 15), 3, False),
                                               ((64, 21, 9), 3, False), ((68, 10, 9), 2, False), ((90, 11, 8), 3, False),
                                               ((20, 20, 20), 4, True), ((62, 62, 62), 1, True)])
@pytest.mark.parametrize("ty", [0, 3, 7, 8, 11])
def test_fp32_row_pairs_match_single_rows(shape, ns, periodic, ty):
    print(f"[case] row pairs {shape} ns={ns} periodic={periodic} ty={ty}", flush=True)
    sd = box(shape, ns, periodic)
    block = 256 if 12 * shape[0] + (12 * max(ty, 16) if periodic else 0) <= 1024 else 512
    if shape[0] * ty > 2 * block:
        ty = 2 * block // shape[0]
    out = []
    for rows in (1, ty):
        with xls.Subdomain(sd, filter_prec=xls.XLS_PREC_FP32) as s:
            s.xls_subdomain_tune(xls.XLS_PREC_FP32, block, rows, 0, 2)
            s.xls_subdomain_filter(3, -3.0, 4.0, 45.0)
            out.append(s.xls_subdomain_get_block())
    assert np.array_equal(out[0], out[1])


# rows of even and odd length, three points a row, a half pair at the end of
# the last row of the box, periodic rows, halo entries past one per lane, tiles
# that fill their lanes and a short last tile
@pytest.mark.parametrize("shape,ns,periodic", [((46, 23, 7), 3, False), ((47, 23, 7), 3, False), ((3, 100, 5), 2, False),
                                               ((17, 21, 14), 4, False), ((24, 24, 24), 3, True), ((64, 16, 9), 2, False),
                                               ((67, 13, 15), 2, False), ((90, 11, 8), 3, False), ((101, 9, 6), 2, False)])
@pytest.mark.parametrize("rows", [0, 1])
def test_fp64_x_pairs_match_single_points(shape, ns, periodic, rows):
    print(f"[case] x pairs {shape} ns={ns} periodic={periodic} rows={rows}", flush=True)
    sd = box(shape, ns, periodic)
    block = 256 if shape[0] <= 80 else 512
    ty = min(shape[1], block // ((shape[0] + 1) // 2)) - rows
    X = np.random.default_rng(6).standard_normal((sd.nd, ns))
    out = []
    for band in (min(ty, max(1, block // shape[0])), ty):  # at most one point a lane, then pairs
        with xls.Subdomain(sd) as s:
            s.xls_subdomain_set_block(X)
            s.xls_subdomain_tune(xls.XLS_PREC_FP64, block, band, 4, 1)
            s.xls_subdomain_filter(3, -3.0, 4.0, 45.0)
            out.append((s.xls_subdomain_get_block(), s.xls_hamiltonian_apply(X)))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])


# Pairs of rows are taken where a row is whole 128-byte lines (nx 32, 64, 96) and
# a lane holds two points: bands of odd and even height whose last one is odd,
# even or a single row, periodic rows (the wrapped partner row, halo columns),
# three and four halo cells a lane, both workgroup sizes and LDS row lengths, one
# and two columns a tile, and the two steps that read a binary16 start
@pytest.mark.parametrize("shape,block,periodic", [((32, 21, 9), 256, False), ((32, 32, 32), 256, True),
                                                  ((64, 21, 9), 256, False), ((64, 23, 15), 512, False),
                                                  ((64, 64, 64), 512, True), ((96, 33, 8), 512, False)])
@pytest.mark.parametrize("nv", [1, 2])
@pytest.mark.parametrize("half", [False, True])
def test_paired_rows_match_one_row_a_lane(shape, block, periodic, nv, half):
    import torch
    sd = box(shape, 3, periodic)
    X = np.random.default_rng(8).standard_normal((sd.nd, 3))
    warm = torch.from_numpy(np.ascontiguousarray(X.T)).half().cuda()
    bands = [ty for ty in range(2, 17) if 1 < shape[0] * ty / block <= 2 and (ty + 1) // 2 * shape[0] <= block]
    assert any(ty % 2 for ty in bands) and any(ty % 2 == 0 for ty in bands)
    ref = None
    for ty in [1] + bands:
        print(f"[case] paired rows {shape} block={block} periodic={periodic} nv={nv} half={half} ty={ty}", flush=True)
        with xls.Subdomain(sd, filter_prec=xls.XLS_PREC_FP32) as s:
            s.xls_subdomain_tune(xls.XLS_PREC_FP32, block, ty, 0, nv)
            if half:
                s.xls_subdomain_use_half(warm)
            else:
                s.xls_subdomain_set_block(X)
            s.xls_subdomain_filter(3, -3.0, 4.0, 45.0)
            got = s.xls_subdomain_get_block()
        ref = got if ref is None else ref
        assert np.array_equal(got, ref)
