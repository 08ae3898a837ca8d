"""The test hooks in icv_conv_params.plan above the public bits: they force a tile or a pipeline shape of the
tensor-core kernels, so that every one of them also runs on problems small enough for the CPU oracle."""

TILES = ["128x64_c2x2", "128x128_c2x2", "256x64_c4x1", "256x64_c4x2", "64x64_c2x2", "256x128_c4x2", "128x128_c4x2"]
GATHER_TILES = (0, 1, 3, 4)          # tiles the gathering kernel (and the plain GEMM) is built for


def tile(index: int) -> int:
    return (index + 1) << 8


def ring(depth: int) -> int:
    return depth << 12


def per_cu(n: int) -> int:
    return n << 16


KCB64 = 1 << 18


def group(taps: int) -> int:
    return taps << 20


# neither a split-reduction kernel nor the window kernel nor, for aligned rows, the any-channel-count one: the plan's own kernel
NO_SPLIT = tile(14)
ANY = tile(12)           # the any-channel-count kernel, whatever the rows, at any number of output pixels


def family(name: str) -> str:
    """The kernel a plan name stands for (icv.h lists the names)."""
    for f in ("window_split", "window", "split", "any", "lowc", "freg", "patch"):
        if f in name:
            return f
    return {"gene": "vector_alu", "gemm": "gemm", "mfma": "gather"}[name[:4]]
