"""The library's real launch code on the CPU, over a recording HIP runtime
(tests/hostsim/fake_runtime.cpp): every entry point runs once with all its
launches and copies succeeding, then once for each of them failing, and must
report the failure each time; and the attention's grid covers every split plan
that the kernel can derive, with little to spare."""
from __future__ import annotations

import ctypes as C
import mmap
import os
import random
import struct
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "hostsim"))
sys.path.insert(0, os.path.dirname(HERE))

import build as hostsim_build  # noqa: E402  (tests/hostsim/build.py)
from paper_2607_00760_amd import _lib  # noqa: E402

OK, HIP = 0, -5


class Sim:
    def __init__(self):
        self.L = _lib.bind_signatures(C.CDLL(hostsim_build.build_launches()))
        self.L.fake_call_name.restype = C.c_char_p
        self.keep = []
        raw = C.create_string_buffer(1 << 16)
        self.keep.append(raw)
        self.any = C.c_void_p((C.addressof(raw) + 255) // 256 * 256)      # stands for device arrays (never read)

    def calls(self):
        """(kernel name, grid) of every recorded call."""
        out, g = [], (C.c_uint * 3)()
        for i in range(self.L.fake_calls()):
            self.L.fake_call_grid(i, g)
            out.append((self.L.fake_call_name(i).decode(), tuple(g)))
        return out

    def cache(self, lens, capacity=None, rotated=1, **kw):
        """A bound cache and its parameters (host memory for the arena)."""
        p = _lib.MosaicParams()
        self.L.mosaic_params_default(C.byref(p))
        for k, v in kw.items():
            if isinstance(v, tuple):
                for i, x in enumerate(v):
                    getattr(p, k)[i] = x
            else:
                setattr(p, k, v)
        h, n = C.c_void_p(), C.c_size_t()
        caps = capacity or max(lens)
        if isinstance(caps, int):
            assert self.L.mosaic_cache_create(C.byref(p), len(lens), caps, rotated, C.byref(h)) == OK
        else:
            assert self.L.mosaic_cache_create_ragged(C.byref(p), len(lens), (C.c_int32 * len(caps))(*caps), rotated, C.byref(h)) == OK
        assert self.L.mosaic_cache_arena_bytes(h, C.byref(n)) == OK
        raw = mmap.mmap(-1, n.value + 4096)                 # (page-aligned, and only touched pages take memory)
        arena = C.addressof(C.c_char.from_buffer(raw))
        assert self.L.mosaic_cache_bind(h, C.c_void_p(arena), n.value) == OK
        self.keep = self.keep[:1] + [raw]
        return dict(h=h, p=p, lens=lens, rotated=rotated, arena=arena)

    def compress(self, c, ws=False):
        n, rot = C.c_size_t(), self.any if c["rotated"] else None
        assert self.L.mosaic_workspace_bytes(c["h"], 0, C.byref(n)) == OK
        return self.L.mosaic_compress(c["h"], self.any, self.any, max(max(c["lens"]), 1),
                                      (C.c_int32 * len(c["lens"]))(*c["lens"]), rot, rot, self.any if ws else None,
                                      n.value if ws else 0, None)

    def decode(self, c):
        n = C.c_size_t()
        assert self.L.mosaic_workspace_bytes(c["h"], 2, C.byref(n)) == OK
        return self.L.mosaic_decode_attention(c["h"], self.any, self.any, C.c_float(0.1), self.any, n.value, None)


@pytest.fixture(scope="module")
def sim():
    return Sim()


OTHER = dict(keep_cand=(24, 40, 64), default_keep=40)            # kept counts of the general encoding kernel


def _compressing(ws, **kw):
    def scenario(s):
        c = s.cache([200, 64, 31], num_kv_heads=2, rot_window=128, **kw)
        return c, lambda: s.compress(c, ws)
    return scenario


def _after_compress(lens, call, **kw):
    def scenario(s):
        c = s.cache(lens, **kw)
        assert s.compress(c) == OK
        return c, lambda: call(s, c)
    return scenario


def _append(s, c):
    return s.L.mosaic_append(c["h"], s.any, s.any, None)


def _closed_window(s, c):
    """The device state after a window of two segments closed on its loss, as the poll reads it."""
    lay = _lib.MosaicLayout()
    assert s.L.mosaic_cache_layout(c["h"], C.byref(lay)) == OK
    for p in range(lay.num_pairs):
        at = c["arena"] + lay.meta_off + p * lay.meta_stride
        C.memmove(at, struct.pack("<iiIIifi", 160, 32, 0, 0, 2, 0.0, 0), 28)
        C.memmove(at + 64, struct.pack("<ii", 0, 2), 8)
    out, n = (C.c_int32 * (3 * lay.num_pairs))(), C.c_int32()
    assert s.L.mosaic_window_poll(c["h"], out, C.byref(n), None) == OK and n.value == lay.num_pairs


def _closing(call, **kw):
    def scenario(s):
        c = s.cache([160, 160], capacity=1000, num_kv_heads=1, rot_window=512, dyn_windows=1, min_window=128, **kw)
        assert s.compress(c) == OK
        _closed_window(s, c)
        return c, lambda: call(s, c)
    return scenario


def _close(s, c):
    return s.L.mosaic_window_close(c["h"], s.any, s.any, s.any, s.any, 128, None)


def _window_rotations(s, c):
    n = C.c_size_t()
    assert s.L.mosaic_workspace_bytes(c["h"], 3, C.byref(n)) == OK
    return s.L.mosaic_window_rotations(c["h"], s.any, s.any, s.any, n.value, None)


def _dense(dtype, group):
    def scenario(s):
        n = C.c_size_t()
        assert s.L.mosaic_dense_workspace_bytes(2, 2, group, 3000, C.byref(n)) == OK
        return None, lambda: s.L.mosaic_dense_decode_attention(s.any, s.any, s.any, s.any, 2, 2, group, 128, dtype, 3000, 3000,
                                                               s.any, C.c_float(0.1), s.any, n.value, None)
    return scenario


def _rotations(reorder):
    def scenario(s):
        p, n, lens = _lib.MosaicParams(), C.c_size_t(), (C.c_int32 * 2)(5000, 70)
        s.L.mosaic_params_default(C.byref(p))
        p.rot_window = 4096
        if reorder:
            assert s.L.mosaic_reorder_workspace_bytes(C.byref(p), 2, 5000, C.byref(n)) == OK
            return None, lambda: s.L.mosaic_reorder_rotations(C.byref(p), 2, 5000, s.any, s.any, 5000, lens, s.any, s.any, s.any,
                                                              n.value, None)
        assert s.L.mosaic_rotation_workspace_bytes(C.byref(p), 2, 5000, C.byref(n)) == OK
        return None, lambda: s.L.mosaic_compute_rotations(C.byref(p), 2, 5000, s.any, s.any, 5000, lens, s.any, s.any, None, None,
                                                          s.any, n.value, None)
    return scenario


SCENARIOS = {
    "compress_two_passes": _compressing(False), "compress_single_pass": _compressing(True),
    "compress_two_passes_other_counts": _compressing(False, **OTHER), "compress_single_pass_other_counts": _compressing(True, **OTHER),
    "append": _after_compress([10], _append, capacity=40), "append_flush": _after_compress([31], _append, capacity=40),
    "append_finalize": _after_compress([63], _append, capacity=70),
    "append_finalize_dyn": _after_compress([63], _append, capacity=300, dyn_windows=1, min_window=64, rot_window=256),
    "decode_short": _after_compress([1000, 500], Sim.decode), "decode_batch": _after_compress([9000] * 4, Sim.decode),
    "decode_bf16_g8": _after_compress([9000], Sim.decode, dtype=1, group_size=8),
    "decode_two_windows": _after_compress([1000], Sim.decode, rot_window=512),
    "decode_many_windows": _after_compress([1200], Sim.decode, rot_window=64),
    "decode_other_counts": _after_compress([9000], Sim.decode, **OTHER),
    "decode_long": _after_compress([132000], Sim.decode, num_kv_heads=1),
    "decode_empty": _after_compress([0], Sim.decode, capacity=100),
    "window_close": _closing(_close), "window_close_other_counts": _closing(_close, **OTHER),
    "window_rotations": _closing(_window_rotations),
    "dense_fp16": _dense(0, 4), "dense_bf16_g8": _dense(1, 8),
    "rotations": _rotations(False), "reorder": _rotations(True),
}


@pytest.mark.parametrize("name", list(SCENARIOS))
def test_every_failed_launch_is_reported(sim, name):
    def once(fail):
        sim.L.fake_reset(-1)
        c, call = SCENARIOS[name](sim)
        sim.L.fake_reset(fail)
        st, calls, message = call(), sim.calls(), sim.L.mosaic_last_error()
        if c:
            assert sim.L.mosaic_cache_destroy(c["h"]) == OK
        return st, calls, message
    st, calls, _ = once(-1)
    assert st == OK and calls
    for i, (what, _) in enumerate(calls):
        st, _, message = once(i)
        assert st == HIP and message, f"{name}: call {i} ({what}) failed, status {st}"


def test_front_kernel_takes_short_contexts_of_up_to_a_pair_per_compute_unit(sim):
    for lens, hkv, want in (([1000] * 32, 8, True), ([40] * 256, 1, True), ([1000] * 33, 8, False), ([40] * 257, 1, False),
                            ([8192], 8, True), ([8224], 8, False)):
        sim.L.fake_reset(-1)
        c = sim.cache(lens, num_kv_heads=hkv)
        assert sim.compress(c) == OK
        sim.L.fake_reset(-1)
        assert sim.decode(c) == OK
        names = [what for what, _ in sim.calls()]
        assert sim.L.mosaic_cache_destroy(c["h"]) == OK
        assert any("k_front" in x for x in names) == want, (lens[:1], len(lens), names)
        assert any("k_topk" in x for x in names) != want


def test_combine_of_two_windows_is_one_kernel_while_its_workgroups_fit_two_rounds(sim):
    # groups of up to four heads always; of eight at most 512 workgroups of 16 columns, 64 pairs
    for group, seqs, W, want in ((4, 9, 128, True), (8, 8, 128, True), (8, 9, 128, False), (5, 16, 128, False), (8, 16, 256, True),
                                 (4, 2, 64, False)):
        sim.L.fake_reset(-1)
        c = sim.cache([250] * seqs, num_kv_heads=8, group_size=group, rot_window=W)
        assert sim.compress(c) == OK
        sim.L.fake_reset(-1)
        assert sim.decode(c) == OK
        names = [what for what, _ in sim.calls()]
        assert sim.L.mosaic_cache_destroy(c["h"]) == OK
        assert any("k_merge" in x for x in names) != want, (group, seqs, W, names)


# ---------------------------------------------------------------- the attention's grid
SLOTS, SPLIT_MIN, SPLIT_MAX, SPLIT_FINE, SPLIT_LEAST = 1024, 48, 128, 16, 8     # 256 CUs, 4 workgroups each


def _splits_of_plan(small, lens, windows, max_sel, max_splits, split_min):
    """The number of splits that the attention's plan makes of these selected
    entries per window of each pair (windows[p]), update buffers included."""
    kt = sum(sum(n) for n in windows)
    buffers = sum(1 for L in lens if L % 64 - (32 if L % 64 >= 32 else 0) > 0)
    et = buffers + sum(1 for n in windows for x in n if x)
    avail = max(SLOTS - et, SLOTS // 4)
    if small:
        tokens = sum(L // 32 for L in lens) * 32 / 10
        b128 = int(128 * kt / max(tokens, 1) + 0.5)
        fit = -(-max(sum(n) for n in windows) * split_min // max_sel)
        rounds = -(-kt // (avail * SPLIT_MAX))
        room = rounds * SLOTS - min(et, SLOTS) if rounds > 1 else avail
        bps = min(max(-(-kt // room), fit, min(max(b128, SPLIT_LEAST), SPLIT_MIN)), SPLIT_MAX)
    else:
        bps = min(max(-(-kt // avail), SPLIT_MIN), SPLIT_MAX)
    return buffers + sum(-(-x // bps) for n in windows for x in n)


# lengths, kv heads, rotation window: both plans, one or more rounds, even and uneven lengths
GRIDS = {
    "batch_two_windows": ([32768] * 4, 8, 16384), "long_batch": ([131072] * 8, 8, 65536), "long_one": ([1 << 20], 8, 65536),
    "long_one_room": ([(1 << 20) + 64], 8, 65536), "uneven_many": ([60000] + [500] * 31, 8, 65536),
    "uneven_many_two_windows": ([100000] + [100] * 31, 8, 65536), "at_128_pairs": ([9000 + 70 * i for i in range(32)], 4, 4096),
    "past_128_pairs": ([9000 + 70 * i for i in range(33)], 4, 4096), "windows_16": ([16000], 8, 1024), "windows_17": ([17000], 8, 1024),
    "short_many": ([40 + i for i in range(64)], 8, 64), "short_133_pairs": ([600 - i for i in range(33)], 4, 448), "short_few": ([1000, 333], 2, 512),
}


@pytest.mark.parametrize("name", list(GRIDS))
def test_attention_grid_covers_the_plan_and_little_more(sim, name):
    lens, hkv, W = GRIDS[name]
    sim.L.fake_reset(-1)
    c = sim.cache(lens, rot_window=W, num_kv_heads=hkv)
    lay = _lib.MosaicWsLayout()
    assert sim.L.mosaic_decode_ws_layout(c["h"], C.byref(lay)) == OK
    assert sim.compress(c) == OK
    sim.L.fake_reset(-1)
    assert sim.decode(c) == OK
    grid = next(g[0] for what, g in sim.calls() if "k_attn" in what)
    assert sim.L.mosaic_cache_destroy(c["h"]) == OK
    nw, npairs = -(-max(lens) // W), len(lens) * hkv
    small = npairs <= 128 and nw <= 16
    desc = max(lens) // 64 + 2
    max_sel = min(16 * desc, -(-(-(-desc * 64 // 10)) // 4) + 1)
    split_min = next(m for m in (SPLIT_MIN, SPLIT_FINE) if lay.max_splits == -(-max_sel // m) + nw + 1)
    pair_lens = [L for L in lens for _ in range(hkv)]
    rng = random.Random(name)
    for blocks in (4, 8, 16, 0):                             # tokens of a block; 0: any number of entries
        for _ in range(20):
            windows = []
            for L in pair_lens:
                k = rng.randint(0, max_sel) if blocks == 0 else min(max_sel, -(-L // 10 // blocks))
                cut = sorted(rng.randint(0, k) for _ in range(nw - 1))
                windows.append([b - a for a, b in zip([0] + cut, cut + [k])])
            need = _splits_of_plan(small, pair_lens, windows, max_sel, lay.max_splits, split_min)
            assert need <= grid, f"{name}: {need} splits for {grid} workgroups"
    # what a plan of this call can need: its rounds of resident workgroups (the
    # general plan: one, or splits of the largest size), a rounding split for
    # every window and buffer
    extra = npairs * (nw + 1)
    full = npairs * -(-max_sel // SPLIT_MAX)
    rounds = -(-full // max(SLOTS - extra, SLOTS // 4)) if small else 1
    assert grid <= max(rounds * SLOTS, 0 if small else full) + extra, f"{name}: {grid} workgroups"
    # and its splits' least size
    assert grid <= npairs * -(-max_sel // (SPLIT_LEAST if small else SPLIT_MIN)) + extra, f"{name}: {grid} workgroups"
