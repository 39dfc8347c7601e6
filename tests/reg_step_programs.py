"""Programs and call sizes that reach the register steps of complex64 dense
passes on tiles below 2^12 amplitudes and with a matrix set per shot; shared by
the test that runs them and the one that looks at which kernels they launch."""
import workloads as W

# 16400 classical bits: more than a resident shot's LDS holds
WIDE_BITS = "bit[16400] wide;\n"


def narrow(n, layers):
    """n = 10, 11 or 12: a state of one tile, off the resident path by its bits."""
    src = W.c1_program(seed=10 * n + layers, n=n, layers=layers, sites=(1, 2), final_measure=False)
    return src.replace("qubit[", WIDE_BITS + "qubit[", 1)


NARROW = [(n, layers) for n in (10, 11, 12) for layers in (3, 24)]
# four tiles and more per resident workgroup (64, 128 and 256 threads of 128
# registers: at most 16, 8 and 4 a CU of 256)
NARROW_SHOTS = {10: 20000, 11: 10000, 12: 10000}


def noisy(n):
    return W.c2_program(seed=5, n=n, layers=6)


NOISY = [13, 14]
NOISY_SHOTS = {13: 2100, 14: 1100}   # 4200 and 4400 tiles: four per workgroup (at most four a CU) and more
NOISY_RATE = 0.01
