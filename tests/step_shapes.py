"""The forecast planner (host code of the library, called without a GPU) and the problems that
reach every shape of block it hands out."""
import ctypes
import random

from paper_2308_03972_amd import binding

MOST = 6


class Dims(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("nx", "ny", "members")]


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("steps", "rx", "ry", "members", "items")]


class Plans(ctypes.Structure):
    _fields_ = [("most", ctypes.c_int), ("fewest", ctypes.c_int), ("p", Plan * (MOST + 1)),
                ("us", ctypes.c_double * (MOST + 1))]


def planner():
    """(step_plans(nx, ny, members, storage), plan_launches(plans, steps, even))."""
    lib = binding.load()
    plans = lib._ZN8lbmletkf10step_plansENS_7LbmDimsEi
    plans.argtypes, plans.restype = [Dims, ctypes.c_int], Plans
    launches = lib._ZN8lbmletkf13plan_launchesERKNS_9StepPlansEib
    launches.argtypes = [ctypes.POINTER(Plans), ctypes.c_int, ctypes.c_bool]
    launches.restype = ctypes.c_int
    return (lambda nx, ny, m, storage: plans(Dims(nx, ny, m), storage),
            lambda p, steps, even: launches(ctypes.byref(p), steps, even))


def shapes(plans):
    """{(steps, members per block, items per thread)} of one problem's launches."""
    return {(n, plans.p[n].members, plans.p[n].items) for n in range(2, plans.most + 1)
            if plans.us[n] < 1e29}


def sample(count, seed):
    """Problems of 1 to 64 members on ragged grids, 10 to 2e7 node-members."""
    rng = random.Random(seed)
    while count:
        m = rng.randint(1, 64)
        p = 10 ** rng.uniform(1, 7.3)
        nx = max(3, int((p / m) ** 0.5 * rng.uniform(0.6, 1.6)))
        ny = max(3, int(p / m / nx))
        if nx <= 2048 and ny <= 2048:
            yield nx, ny, m, rng.randint(0, 1)
            count -= 1


# (nx, ny, members, storage): small problems that between them have every (storage, members per
# block, items per thread) of the planner: 1 to 12 members in FP64, 1 to 5 and 7 to 12 in FP32
REACH = [(nx, ny, m, 0) for nx, ny, m in
         [(4, 3, 1), (495, 257, 1), (22, 12, 19), (167, 110, 5), (95, 44, 3), (256, 166, 3),
          (13, 11, 46), (94, 38, 44), (67, 37, 5), (102, 269, 5), (153, 108, 12), (55, 41, 13),
          (71, 180, 14), (57, 50, 16), (188, 201, 15), (73, 30, 17), (115, 145, 18), (67, 63, 19),
          (141, 89, 19), (31, 72, 22), (101, 122, 21), (67, 89, 23), (195, 92, 24)]]
REACH += [(nx, ny, m, 1) for nx, ny, m in
          [(3, 3, 1), (7, 13, 55), (3, 3, 2), (17, 10, 59), (60, 62, 3), (42, 60, 8), (27, 13, 43),
           (70, 42, 15), (26, 11, 51), (112, 89, 13), (86, 42, 13), (90, 48, 24), (239, 169, 8),
           (215, 99, 17), (56, 41, 17), (136, 123, 60), (70, 163, 19), (67, 88, 21), (92, 45, 21),
           (55, 44, 23)]]
