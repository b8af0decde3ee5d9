"""Builds of the library for the tests of csrc/part_exchange.h: workgroups that give up on the others' words at once ("never"), or on a
pseudo-random quarter of them ("some": some words there and others not, statistics there and masses missing), and compute
what is missing themselves. The name of a build has the digest of what it was made from: one of other sources is not used."""
import glob
import os

from paper_2503_05096_amd import build

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")
DEFINES = {
    "never": ["ADASPEC_PATIENCE(word)=0"],
    # a hash of (workgroup, word)
    "some": ["ADASPEC_PATIENCE(word)=((((unsigned)((unsigned long long)(word)>>3)+blockIdx.x*40503u)*2654435761u>>15&3u)?64:0)"],
}


def path(name: str) -> str:
    return os.path.join(NATIVE, f"libadaspec_{name}_{build.source_key(DEFINES[name])}.so")


def ensure(name: str) -> str:
    out = path(name)
    if not os.path.exists(out):
        for old in glob.glob(os.path.join(NATIVE, f"libadaspec_{name}_*.so")):
            os.remove(old)
        made = f"{out}.{os.getpid()}"
        build.build_variant(made, name, DEFINES[name], "part_exchange.h")
        os.replace(made, out)
    return out
