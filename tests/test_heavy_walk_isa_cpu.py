"""The queue claims of the heavy groups' walk in the gfx950 code (CPU only):
as for the main walk (test_walk_isa_cpu.py), every claim is a returning atomic
alone in a one-lane region, closed at once, its result made wave-uniform."""
import test_walk_isa_cpu as W
from test_walk_isa_cpu import asm  # noqa: F401


def test_heavy_walk_claims_are_wave_uniform(asm, monkeypatch):  # noqa: F811
    text = asm.replace("12k_heavy_walkI", "12k_walk_heavyI")
    monkeypatch.setattr(W, "WALK_KERNELS", ("k_walk_heavy",))
    assert len(W.functions(text)) == 8  # compensated x hash x potential
    W.test_queue_claims_are_wave_uniform(text)
