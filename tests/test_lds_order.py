"""Values that lanes of a wave hand each other through LDS (a property of the
sources: which compilers keep an unfenced order cannot be tested)."""

from pathlib import Path

CSRC = Path(__file__).parent.parent / "paper_2408_10154_amd" / "csrc"


def test_wave_barriers_come_with_fences():
    sites = [(p.name, line.strip()) for p in sorted(CSRC.glob("*")) if p.suffix in (".hip", ".h")
             for line in p.read_text().splitlines() if "wave_barrier()" in line]
    assert sites == [("common.h", "__builtin_amdgcn_wave_barrier();")]  # in wave_sync
