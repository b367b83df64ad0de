"""Properties of the built kernels that their speed rests on and that a
change elsewhere can take away unseen: how the persistent batch reads its
frame tables."""
import kernelcode


def test_persistent_batch_reads_its_tables_by_scalar_loads():
    """A frame's fields come through the constant address space.  Flat loads
    mean that a table, or a pointer from one, is read as ordinary memory:
    every lane then loads every field again after each fence (24 uneven SSGI
    frames 3.9 ms instead of 2.5)."""
    counts = kernelcode.instructions("k_fused.hip")
    flat = sum(n for op, n in counts.items() if op.startswith("flat_load"))
    scalar = sum(n for op, n in counts.items() if op.startswith("s_load"))
    assert scalar > 0 and flat == 0, (scalar, flat)
