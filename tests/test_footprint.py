"""pf_footprint_bytes of reducing and spectral models (no GPU)."""
import paper_2511_10508_amd as P


def test_footprint_counts_reduction_partials():
    """The partials of many steps, one pair per wave and quantity: more than 256 steps
    of a small grid's at least, 32 MiB and the finalising level (a quarter of that)
    at most."""
    for n in ((128, 128), (256, 256), (1024, 1024), (64, 64, 64)):
        plain = P.footprint_bytes(P.make_desc(P.PF_CH, n, dt=1e-3))
        red = P.footprint_bytes(P.make_desc(P.PF_CH, n, dt=1e-3, flags=P.PF_REDUCE_EACH_STEP))
        assert 256 * 3 * 16 * 4 <= red - plain <= (32 << 20) * 5 // 4, n


def test_footprint_counts_padded_spectra_and_twiddles():
    """Power-of-two spectral grids: half spectra padded to groups of 64 bytes, FP64
    twiddle tables."""
    for prec, eb, cols in ((P.PF_FP64, 8, 36), (P.PF_FP32, 4, 40)):
        plain = P.footprint_bytes(P.make_desc(P.PF_AC, (64, 32), dt=1e-3, precision=prec))
        spec = P.footprint_bytes(P.make_desc(P.PF_AC, (64, 32), dt=1e-3, precision=prec, flags=P.PF_SPECTRAL))
        assert spec == plain + 2 * cols * 32 * 2 * eb + 16 * (64 + 32)
