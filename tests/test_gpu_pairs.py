"""GPU: the radix-pair line kernels at every compiled radix and at the edges of their ranges.

Thin boxes whose long edge runs through the lengths below along x, y and z: every radix of
either stage of the direct pairs, the chirp-z lengths around the class limits (padded
lengths up to 576 and up to 1024), and the first lengths past them, which stay on the
Stockham kernels.  One push of random fields against the oracle (FP64 <= 1e-12 relative,
FP32 <= 2e-5 relative, max norm: about log2 N rounding errors of 6e-8 per transform).
"""

import numpy as np
import pytest

import synth
from oracle import step

pytestmark = pytest.mark.gpu

# direct: 1..18 and 20, 21, 22, 24 alone, then products that reach each stage B and class 1 radix
DIRECT = list(range(1, 19)) + [20, 21, 22, 24, 24 * 2, 24 * 3, 22 * 5, 21 * 7, 20 * 9, 18 * 11, 24 * 13, 22 * 17,
                               21 * 15, 22 * 21, 24 * 24, 25 * 24, 27 * 26, 28 * 12, 30 * 28, 32 * 17, 33 * 32,
                               34 * 33, 36 * 36]
# chirp-z: padded lengths 2n - 1 <= 16 .. 576 (class of small radices) and .. 1024, odd and even n
CHIRP = [19, 23, 38, 46, 53, 74, 101, 134, 199, 202, 254, 283, 286, 307, 446, 509]
# smooth without a pair, and chirp-z beyond 1024 padded points
STOCKHAM = [245, 343, 521]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_every_pair_length_matches_oracle(lib, axis, precision):
    import torch

    for n in DIRECT + CHIRP + STOCKHAM:
        if axis == 2 and precision == "fp64" and lib.default_schedule(n)[1] > 850:
            continue  # eleven FP64 z lines of that length exceed a workgroup's LDS: refused
        edges = [5, 5]  # odd: a ragged pair of rows in the x passes, a ragged last tile elsewhere
        edges.insert(axis, n)
        plan = lib.Plan(*edges, nguard=0, order=8, dx=1.0, dt=0.5, precision=precision)
        f = synth.random_fields(synth.rng_for(210 + axis, n), plan.box_shape)
        ref = step.box_step(f, 1.0, 0.5, 8)
        print(f"pair box {edges} {precision} {plan.schedule(axis)}", flush=True)
        g = torch.as_tensor(f, dtype=plan.dtype, device="cuda")
        plan.push_fields(g)
        torch.cuda.synchronize()
        err = np.abs(g[0:6].double().cpu().numpy() - ref).max() / np.abs(ref).max()
        assert err <= (1e-12 if precision == "fp64" else 2e-5), (edges, err)
        plan.close()


def test_batch_of_direct_and_chirp_boxes_equals_single_boxes(lib):
    """Boxes of different radix pairs, chirp-z lengths and one without a pair in one batch: every
    box bitwise as its own plan (the same line transforms)."""
    import torch

    gdims = (160, 70, 64)
    boxes = [dict(origin=(0, 0, 0), interior=(40, 37, 30), nguard=(7, 8, 4), order=8),      # 54 x 53 x 38
             dict(origin=(40, 0, 0), interior=(61, 37, 64), nguard=(20, 2, 0), order=16),   # 101 x 41 x 64
             dict(origin=(101, 0, 0), interior=(59, 37, 64), nguard=(93, 6, 8), order=0),   # 245 x 49 x 80
             dict(origin=(0, 37, 0), interior=(160, 33, 64), nguard=(8, 5, 3), order=4)]    # 176 x 43 x 70
    g1 = torch.as_tensor(synth.random_fields(synth.rng_for(213, 0), gdims[::-1]), dtype=torch.float32, device="cuda")
    batch = lib.Batch(boxes, gdims, dt=0.5)
    got = g1.clone()
    batch.step(got)
    for b in boxes:
        plan = lib.Plan(*b["interior"], nguard=b["nguard"], order=b["order"], dt=0.5)
        one = g1.clone()
        plan.step_g1(one, b["origin"])
        (ox, oy, oz), (nx, ny, nz) = b["origin"], b["interior"]
        at = (slice(0, 6), slice(oz, oz + nz), slice(oy, oy + ny), slice(ox, ox + nx))
        torch.cuda.synchronize()
        assert torch.equal(got[at], one[at]), plan.box
        plan.close()
    batch.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx", [24, 600, 38, 311, 245])
def test_odd_boxes_read_nothing_outside_them(lib, nx, precision):
    """The last row of an odd box has no partner: whatever the cells outside the box hold, its fields are
    the same bit for bit (direct, chirp-z and Stockham x lines; alone and in a batch)."""
    import torch

    dtype = torch.float64 if precision == "fp64" else torch.float32
    box = dict(origin=(5, 7, 6), interior=(nx - 4, 9, 7), nguard=2, order=8)   # nx x 13 x 11 cells
    gdims = (nx + 12, 40, 24)
    f = torch.as_tensor(synth.random_fields(synth.rng_for(214, nx), gdims[::-1]), dtype=dtype, device="cuda")
    covered = torch.zeros(gdims[::-1], dtype=torch.bool, device="cuda")
    covered[4:15, 5:18, 3:3 + nx] = True
    plan = lib.Plan(*box["interior"], nguard=2, order=8, dt=0.5, precision=precision)
    batch = lib.Batch([box], gdims, dt=0.5, precision=precision)
    at = (slice(0, 6), slice(6, 13), slice(7, 16), slice(5, 1 + nx))
    for name, advance in (("plan", lambda g: plan.step_g1(g, box["origin"])), ("batch", batch.step)):
        out = []
        for outside in (0.0, float("nan")):
            g = torch.where(covered, f, torch.full_like(f, outside))
            advance(g)
            torch.cuda.synchronize()
            out.append(g[at].clone())
        assert torch.isfinite(out[1]).all(), name
        assert torch.equal(out[0], out[1]), name
    plan.close()
    batch.close()


# lengths with a pair that the Stockham kernels beat on at least one axis, and their neighbours that keep it
EITHER = [17, 34, 51, 125, 175, 241, 243, 250, 256, 257, 363, 390, 429, 495, 510, 512, 561, 612, 714]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_lengths_that_keep_the_stockham_kernels_match_oracle(lib, axis, precision):
    import torch

    kinds = set()
    for n in EITHER:
        edges = [7, 5]
        edges.insert(axis, n)
        plan = lib.Plan(*edges, nguard=0, order=8, dx=1.0, dt=0.5, precision=precision)
        kinds.add(bool(plan.query(lib.Q_TWO_STAGE) >> (0, 1, 2)[axis] & 1))
        f = synth.random_fields(synth.rng_for(215 + axis, n), plan.box_shape)
        ref = step.box_step(f, 1.0, 0.5, 8)
        g = torch.as_tensor(f, dtype=plan.dtype, device="cuda")
        plan.push_fields(g)
        torch.cuda.synchronize()
        err = np.abs(g[0:6].double().cpu().numpy() - ref).max() / np.abs(ref).max()
        assert err <= (1e-12 if precision == "fp64" else 2e-5), (edges, err)
        plan.close()
    assert kinds == {True, False}
