"""Properties of the built kernels that their speed rests on and that a
change elsewhere can take away unseen: how the persistent batch reads its
frame tables, and how many waves the launches with depth tiles hold."""
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


def test_depth_tile_launches_hold_eight_waves_per_simd():
    """(Seven for batches with a halo of 24 texels, whose tile and row tables
    share the LDS.)  With five they were slower than gathers from the plane
    by more than the tiles saved."""
    single = {k: kernelcode.waves_per_simd(m) for k, m in kernelcode.kernels("k_ssao.hip").items() if "k_ssao_tiled" in k}
    batch = {k: kernelcode.waves_per_simd(m) for k, m in kernelcode.kernels("k_ssao_tiles.hip").items()}
    assert len(single) == 6 and len(batch) == 6
    assert all(w == 8 for w in single.values()), single
    assert all(w >= (7 if "Li24E" in k else 8) for k, w in batch.items()), batch
