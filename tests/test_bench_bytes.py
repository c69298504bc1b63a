"""The benchmark's byte count of the V-cycle kernels that the profiler does not
bracket: the transfers of the levels above the dense one and its product, nothing
for the coarse residuals, which the sweeps form from entries they hold."""
import numpy as np

import bench


class Lib:
    GL_FP64, GL_FP32 = 0, 1

    def __init__(self, dense_rows):
        self.dense_rows = dense_rows

    def gl_precond_get_tiles(self, pre):
        return {"lane_shift": 0, "bottom_rows": 64, "dense_rows": self.dense_rows, "l0_tiled": 2}


class Pre:
    P = {1: 30, 2: 7}

    def info(self):
        return {"nlev": 4, "sizes": [1000, 100, 20, 5], "nnz": [10 ** 6, 10 ** 7, 10 ** 8, 25], "ncolors": [2, 4, 5, 5]}

    def export(self, level, what):
        assert what == "P_rp"
        return np.array([0, self.P[level]])


def transfers(nf, nc, pn, sz):
    # P and R: values, columns, row pointers; the residual written and read, the
    # coarse right-hand side written, the coarse iterate read
    return 2 * pn * (4 + sz) + 4 * (nf + 1 + nc + 1) * 2 + 2 * (nf + nc) * sz


def test_iteration_bytes():
    for prec, sz in ((Lib.GL_FP64, 16), (Lib.GL_FP32, 8)):
        one = transfers(100, 20, 30, sz)
        assert bench.iteration_bytes(Lib(50), Pre(), prec) == one + 400 * sz + 2 * 20 * sz
        assert bench.iteration_bytes(Lib(0), Pre(), prec) == one + transfers(20, 5, 7, sz) + 25 * sz + 2 * 5 * sz
