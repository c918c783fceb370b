"""Build the test-only libraries of tests/native with the library's compiler
flags: the HIP kernels of fp64 division and square root (libfp64ops.so), and
the library with work-groups that never read the state of another tile
(libtilesums.so, its other objects the library's)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
LIB = os.path.join(HERE, "libfp64ops.so")
TILES_LIB = os.path.join(HERE, "libtilesums.so")
TILED = ("util", "links", "ntuplets", "fishbone")   # sources whose kernels list by tiles


def build(verbose: bool = False) -> str:
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    from paper_2008_13461_amd import build as B
    cmd = [B.HIPCC, *B.FLAGS, "-shared", "-o", LIB + ".tmp", os.path.join(HERE, "fp64_ops.hip")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    build_tiles(B, verbose)
    return LIB


def build_tiles(B, verbose: bool = False) -> str:
    import concurrent.futures as cf

    stems = [s.replace(".hip", "") for s in B.SOURCES]
    objs = os.path.join(B.HERE, "_build")
    if not all(os.path.exists(os.path.join(objs, s + ".o")) for s in stems):
        B.build(verbose)
    own = os.path.join(HERE, "_build")
    os.makedirs(own, exist_ok=True)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with cf.ThreadPoolExecutor(max_workers=len(TILED)) as ex:
        list(ex.map(lambda s: run([B.HIPCC, *B.FLAGS, "-DPT_TILE_POLLS=-1", "-c", os.path.join(B.CSRC, s + ".hip"),
                                   "-o", os.path.join(own, s + ".o")]), TILED))
    run([B.HIPCC, f"--offload-arch={B.ARCH}", "-shared", "-fPIC", "-o", TILES_LIB + ".tmp",
         *(os.path.join(own if s in TILED else objs, s + ".o") for s in stems)])
    os.replace(TILES_LIB + ".tmp", TILES_LIB)
    return TILES_LIB


if __name__ == "__main__":
    build(verbose=True)
