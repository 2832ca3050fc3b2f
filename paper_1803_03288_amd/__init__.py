"""TicTac scheduling math on MI355X: recv-dependency bitsets, TIC/TAC transfer
priorities and batched makespan / scheduling-efficiency evaluation.

Sub-modules
-----------
workloads : seeded synthetic DAG and timing-sample generators (no scheduling
            arithmetic; shared by the tests of the oracle and of the GPU
            path).
binding   : ctypes binding of the C-ABI library (``libtictac.so``) built from
            ``csrc/``; everything per timing sample runs in the HIP kernels, and
            so do the dependency sets of large graphs (those of small ones
            are formed by the library's host code).
build     : compiles ``csrc/`` for gfx950 with hipcc.

Nothing is imported eagerly so that the generator module can be used on a
machine without the compiled library.
"""

__all__ = ["workloads", "binding", "build"]
