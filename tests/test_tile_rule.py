"""The tile shapes of layers that nothing was tuned for: valid for every size
and width, never a split of the reduction (the batch plan, which does not
split, has to equal the single calls bit for bit), and taller for larger
grids.  Host code only: no GPU."""
import ctypes
import os
import subprocess
import sys

import pytest

from paper_2305_11566_amd import _lib


def _names(c, latent, f, dtype, B, H, W):
    d = _lib.make_desc(*c, latent, f, dtype)
    arr = (ctypes.c_int * 9)()
    assert _lib.lib().sv_layer_cfgs(ctypes.byref(d), B, H, W, arr) == 0
    return [_lib.lib().sv_conv_cfg_name(a).decode() for a in arr]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16", "i8"])
@pytest.mark.parametrize("c,latent", [((8, 8, 8), 8), ((16, 32, 64), 64), ((32, 64, 128), 128), ((40, 96, 256), 256)])
def test_every_size_has_an_unsplit_tile(monkeypatch, tmp_path, dtype, c, latent):
    monkeypatch.setenv("SV_AUTOTUNE_CACHE", str(tmp_path / "none.tsv"))
    for f, H, W in ((1, 1, 1), (2, 17, 33), (4, 375, 1242), (2, 256, 512), (8, 2000, 3000)):
        for B in (1, 2, 7, 64, 500):
            for n in _names(c, latent, f, dtype, B, H, W):
                assert n.startswith("th") and "_s" not in n, (n, f, H, W, B)


def test_larger_grids_take_taller_tiles(monkeypatch, tmp_path):
    monkeypatch.setenv("SV_AUTOTUNE_CACHE", str(tmp_path / "none.tsv"))
    rows = [int(_names((32, 64, 128), 128, 4, "bf16", B, 375, 1242)[7][2:].split("_")[0]) for B in (1, 2, 4, 64)]
    assert rows == [4, 8, 16, 16]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16", "i8"])
@pytest.mark.parametrize("c,latent", [((16, 32, 64), 64), ((40, 96, 256), 128)])
def test_tall_tiles_where_few_rows_are_padded(monkeypatch, tmp_path, dtype, c, latent):
    """A tall tile's rows, whole tiles, are at most a third more than four-row (two-row at
    stride 2) tiles would compute: many maps of 9 or 10 rows are no reason for 16."""
    monkeypatch.setenv("SV_AUTOTUNE_CACHE", str(tmp_path / "none.tsv"))
    levels = (1, 2, 3, 3, 3, 2, 1, 0)  # 0: the network's working size, each next one half
    for h in (4, 9, 10, 17, 18, 19, 33, 37, 40, 72, 128):
        ho = [h]
        for _ in range(3):
            ho.append(-(-ho[-1] // 2))
        for B in (1, 8, 64, 300):
            for i, n in enumerate(_names(c, latent, 1, dtype, B, h, 200)[:8]):
                th, rows = int(n[2:].split("_")[0]), ho[levels[i]]
                low = 2 if i in (0, 1, 2) else 4
                if th > 4:
                    assert 3 * -(-rows // th) * th <= 4.1 * -(-rows // low) * low, (n, i, B, h)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16", "i8"])
@pytest.mark.parametrize("c,latent", [((8, 8, 128), 8), ((16, 64, 64), 64), ((40, 96, 256), 128), ((72, 136, 200), 8)])
def test_large_batches_keep_within_a_grid(monkeypatch, tmp_path, dtype, c, latent):
    """Images times channel tiles of a launch are at most 65535: a batch that 64
    channels a tile (or all of a narrower layer's) can take is taken by the rule's."""
    monkeypatch.setenv("SV_AUTOTUNE_CACHE", str(tmp_path / "none.tsv"))
    c1, c2, c3 = c
    cout = (c1, c2, c3, 2 * latent, c3, c2, c1, c1)
    for H, W in ((8, 8), (30, 33), (128, 128)):
        for B in (10000, 16384, 20000, 21846, 32768, 50000, 65535):
            for n, co in zip(_names(c, latent, 1, dtype, B, H, W), cout):
                tn = int(n.split("_tn")[1].split("_")[0])
                if B * -(-co // 64) <= 65535:
                    assert B * -(-co // tn) <= 65535, (n, co, B, H, W)


def _cached(tmp_path, lines, queries):
    """Names for (B, H, W) queries in a process of its own that reads this cache, and its messages."""
    cache = tmp_path / "tune.tsv"
    cache.write_text("".join(l + "\n" for l in lines))
    code = ("import sys; sys.path.insert(0, '.')\n"
            "from tests.test_tile_rule import _names\n"
            f"for q in {queries!r}: print(','.join(_names((32, 64, 128), 128, 4, 'bf16', *q)))\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True,
                       env=dict(os.environ, SV_AUTOTUNE_CACHE=str(cache)))
    assert r.returncode == 0, r.stderr
    return r.stdout.split(), r.stderr


def test_cached_choices(tmp_path):
    """Entries timed on other kernels are passed over without a message; a choice that
    is the rule's at its own batch follows the rule at other batches; any other holds
    to twice and half its batch."""
    key = "dt1|c32,64,128|L128|f4|B%d|375x1242\t4\t%s"
    queries = [(1, 375, 1242), (2, 375, 1242), (64, 375, 1242)]
    rule, err = _cached(tmp_path, [], queries)
    assert len(set(rule)) == 3
    other = ",".join(["th8_tn16_k2"] * 9)
    old = ["gfx950|" + key % (1, other), "gfx950|r1|" + key % (1, other)]
    assert _cached(tmp_path, old, queries) == (rule, err)
    assert _cached(tmp_path, ["gfx950|r2|" + key % (1, rule[0])], queries)[0] == rule
    assert _cached(tmp_path, ["gfx950|r2|" + key % (1, other)], queries)[0] == [other, other, rule[2]]
    out, err = _cached(tmp_path, ["garbage"], queries)
    assert out == rule and "malformed" in err
