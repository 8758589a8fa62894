"""Solves whose steps are taken in pairs (two in one pass over the lattice), for
the GPU tests that compare pairs with single steps and for the CPU test that
checks that they are planned so."""
import workloads as WL

P, W, V, O, ZV, ZO = (WL.PERIODIC, WL.WALL, WL.VELOCITY, WL.PRESSURE, WL.ZH_VELOCITY, WL.ZH_PRESSURE)

FACES = {"periodic": [P] * 6, "channel": [V, O, W, W, P, P], "closed": [W] * 6, "zou_he": [ZV, ZO, W, W, P, P],
         "zou_he_z_walls": [ZO, ZV, P, P, W, W], "duct": [P, P, W, W, W, W], "wall_out": [W, O, P, P, P, P]}

# a last column of one cell (129, 257) and a box narrower than a column (61),
# each with a last tile of one row along z (12 k + 1)
RAGGED = [(129, 97, 133), (257, 97, 49), (61, 200, 205)]


def lattice(size, bc):
    return WL.box(*size, bc, 0.6, u_in=(0.03, 0.002, -0.001) if bc[0] != P else (0, 0, 0), rho_out=1.001)


def foil(case, complete_case):
    """Foils and a body force: completed box and wings."""
    if case == "clap_fling":
        bx, wg, ph = WL.clap_fling_case()
    elif case == "cylinder":
        bx, wg, ph = WL.cylinder_case(nx=257, ny=190, nz=193, d=20.0)
    else:
        bx, wg, ph = WL.plate_case(nx=256, ny=192, nz=192, centre=(60.2, 6.4))
    return complete_case(dict(bx, body_force=[2e-6, -1e-6, 3e-6]), wg, ph)


def batch(complete_case):
    """(box, wings, storage, check interval, first step, steps alone before the
    batch) of solves of one batch: lattices, long and short spans, a foil whose
    neighbours wrap, check steps, 16-bit storage, a body force.  Their windows
    of 64 steps start at different steps, so that after a while first, second
    and single steps are taken together."""
    out = [(lattice((256, 192, 192), FACES["periodic"]), [], "fp32", 0, 0, 0),
           (lattice((130, 61, 97), FACES["zou_he"]), [], "fp32", 0, 0, 3),
           (lattice((129, 64, 97), FACES["closed"]), [], "fp32", 0, 0, 2)]
    for k, (nx, ny, nz, c, sto, check) in enumerate([(64, 48, 8, 8.0, "fp32", 0), (97, 80, 81, 10.0, "fp32", 0),
                                                     (70, 60, 13, 8.0, "fp32", 0), (160, 128, 128, 16.0, "fp32", 0),
                                                     (96, 80, 40, 10.0, "fp32", 5), (64, 48, 16, 8.0, "fp16", 0),
                                                     (128, 96, 60, 12.0, "fp32", 0), (65, 50, 16, 8.0, "fp32", 0)]):
        bx, wg, ph = WL.clap_fling_case(nx=nx, ny=ny, nz=nz, chord=c)
        if k == 6:
            bx = dict(bx, body_force=[2e-6, -1e-6, 3e-6])
        out.append((*complete_case(bx, wg, ph), sto, check, 40 + k, k % 4))
    bx, wg, ph = WL.plate_case(nx=70, ny=40, nz=24, centre=(9.0, 9.5))
    out.append((*complete_case(dict(bx, bc=[P] * 6, u_in=[0.0, 0.0, 0.0]), wg, ph), "fp32", 0, 0, 1))
    return out
