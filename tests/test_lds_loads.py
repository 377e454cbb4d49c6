"""Loads straight into LDS have arrived before that LDS serves something else (tests/lds_loads.py), by the compiled code of a kernel."""
import lds_loads


def test_the_reader_follows_every_path():
    wait, load, store = "s_waitcnt vmcnt(%d)", "global_load_lds_dwordx4 v[0:1], off", "global_store_dword v0, v1, s[0:1]"
    code = lambda *lines: list(enumerate(lines, 1))
    ends = lambda *lines: [l for l in lds_loads.under_way(code(*lines)) if l[1] == "s_endpgm"]
    assert ends(load, "s_endpgm") and not ends(load, wait % 0, "s_endpgm")
    assert ends(load, wait % 1, "s_endpgm") and not ends(load, store, wait % 1, "s_endpgm")
    assert ends(load, "s_cbranch_scc1 .L1", wait % 0, ".L1:", "s_endpgm")                    # the wait is skipped
    assert not ends(load, "s_cbranch_scc1 .L1", store, ".L1:", wait % 0, "s_endpgm")
    assert ends(".L1:", load, store, "s_cbranch_scc1 .L1", wait % 2, "s_endpgm")
    assert not ends("s_branch .L1", load, ".L1:", "s_endpgm")


def test_framed_weight_gradients_exchange_sums_behind_their_loads():
    """Runs of one or two units take the steps of an incomplete chunk alone, past the loop whose waits serve all others."""
    code, = [c for name, c in lds_loads.kernels("hq_wgrad_band.hip").items() if "hq_wgrad_band_kernel" in name]
    assert sum(l.startswith("global_load_lds") for _, l in code) >= 6 and sum(l.startswith("ds_write_b128") for _, l in code) >= 6
    early = [(n, l) for n, l in lds_loads.under_way(code) if l.startswith(("ds_write", "ds_add")) and not l.startswith("ds_write_b8") or l == "s_endpgm"]
    assert not early, early                                   # (the bytes are the position masks, which lie apart)
