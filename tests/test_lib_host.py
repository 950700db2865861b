"""CPU-side checks of the C-ABI library: it loads without a GPU, exports every declared symbol,
and its host-only calls (partition, sizes, layout, argument validation) agree with the oracle."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2107_00961_amd as R
from oracle import partition as OP
from oracle import resnet as OR
from resist_inputs import get_config, make_params

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exports_every_declared_symbol():
    lib = R.lib()
    declared = set()
    for hdr in ("resist.h", "resist_ops.h"):
        src = open(os.path.join(ROOT, "include", hdr)).read()
        src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
        declared |= set(re.findall(r"\b(resist_[a-z0-9_]+)\s*\(", src))
    assert {"resist_partition", "resist_local_step", "resist_aggregate"} <= declared
    for name in declared:
        assert hasattr(lib, name), name


@pytest.mark.parametrize("cfg,S,min_depth", [("cfg1", 1, 0), ("cfg2", 4, 0), ("cfg4", 2, 0), ("cfg2", 8, 5),
                                             ("cfg2", 3, 12), ("cfg2", 16, 0), ("cfg4", 5, 10)])
def test_partition_bit_exact(cfg, S, min_depth):
    model = get_config(cfg)["model"]
    for seed in (0, 1, 2, 12345678901234567890):
        for rnd in (0, 1, 7):
            assert R.partition(model, S, min_depth, seed, rnd) == OP.partition(model["blocks"], S, min_depth, seed, rnd)


def test_partition_paper_mask_and_errors():
    model = get_config("cfg3")["model"]
    nb = R.num_blocks(model)
    mask = [1 if 7 < b < 30 else 0 for b in range(nb)]
    for S, md in ((2, 0), (4, 0), (8, 4)):
        assert R.partition(model, S, md, 3, 2, mask) == OP.partition(model["blocks"], S, md, 3, 2, mask)
    with pytest.raises(R.ResistError):
        R.partition(model, 0, 0, 0, 0)
    with pytest.raises(R.ResistError):
        R.partition(model, 2, -1, 0, 0)
    # capacity error: nothing is written past cap
    d = R.model_desc(model)
    offs = (ctypes.c_int32 * 5)()
    blocks = (ctypes.c_int32 * 8)(*([-7] * 8))
    owner = (ctypes.c_int32 * nb)()
    rc = R.lib().resist_partition(ctypes.byref(d), None, 4, 0, 1, 0, offs, blocks, 8, owner)
    assert rc == -3 and list(blocks) == [-7] * 8
    assert b"cap" in R.lib().resist_last_error()


@pytest.mark.parametrize("cfg", ["cfg1", "cfg2", "cfg3", "cfg4"])
def test_param_counts_and_layout(cfg):
    model = get_config(cfg)["model"]
    nb = R.num_blocks(model)
    assert nb == sum(model["blocks"])
    params = make_params(model, 0, perturb_bn=True)
    for b in range(-1, nb + 1):
        tot, tr = R.block_param_count(model, b)
        lay = R.block_layout(model, b)
        assert sum(t["count"] for t in lay if t["kind"] not in (3, 4)) == OR.param_count(model, b)
        assert sum(t["count"] for t in lay) == OR.param_count(model, b, trainable_only=False)
        assert all(t["offset"] % 4 == 0 for t in lay)
        assert tr <= tot and tr % 4 == 0 and tot % 4 == 0
        ends = [t["offset"] + t["count"] for t in lay]
        assert all(lay[i + 1]["offset"] >= ends[i] for i in range(len(lay) - 1)) and ends[-1] <= tot
        # pack -> unpack is the identity on logical tensors
        flat = R.pack_block(model, b, params[b])
        back = R.unpack_block(model, b, flat)
        assert set(back) == set(params[b])
        for k in back:
            np.testing.assert_array_equal(back[k], params[b][k])


def test_conv_weight_layout_is_krsc():
    model = get_config("cfg1")["model"]
    w = np.arange(16 * 16 * 9, dtype=np.float32).reshape(16, 16, 3, 3)
    flat = R.pack_block(model, 0, {"conv1_w": w})
    k, c, r, s = 5, 7, 2, 1
    assert flat[((k * 3 + r) * 3 + s) * 16 + c] == w[k, c, r, s]


@pytest.mark.parametrize("kind", [0, 2])
def test_workspace_of_a_step_too_small_for_the_second_stream(kind):
    """Below 20 GFLOP a step gets along with two output-gradient buffers: 16 tensors of the activations' size in all, where from there
    up there are four more (1416 images of 14.1 MFLOP)."""
    model = dict(get_config("cfg1")["model"], block_kind=kind)
    act = lambda batch: 4 * batch * 16 * 16 * 16
    small, large = R.workspace_bytes(model, [0, 1], 1410) / act(1410), R.workspace_bytes(model, [0, 1], 1420) / act(1420)
    assert small < 16.5 and 3.9 < large - small < 4.1


def test_workspace_and_step_argument_errors():
    model = get_config("cfg2")["model"]
    with pytest.raises(R.ResistError, match="first block"):
        R.workspace_bytes(model, [0, 1, 2], 8)
    with pytest.raises(R.ResistError, match="ascending"):
        R.workspace_bytes(model, [0, 3, 3, 7, 30], 8)
    with pytest.raises(R.ResistError):
        R.workspace_bytes(model, [0, 3, 7, 30, 99], 8)
    with pytest.raises(R.ResistError):
        R.workspace_bytes(model, [0, 3, 7, 30], 0)
    assert R.workspace_bytes(model, [0, 3, 7, 30], 8) > 0
    bad = dict(model, widths=[60, 128, 256, 512])
    with pytest.raises(R.ResistError, match="multiple of 16"):
        R.num_blocks(bad)
    # NULL buffers are refused before anything is launched (no GPU needed to see the error)
    d = R.model_desc(model)
    blocks = (ctypes.c_int32 * 4)(0, 3, 7, 30)
    rc = R.lib().resist_local_step(ctypes.byref(d), blocks, 4, None, None, None, None, None, 8, 0.1, 0.9, 0.0,
                                   None, 0, None, None)
    assert rc == -1


@pytest.mark.parametrize("kind", [2, 3])
def test_preactivation_layouts(kind):
    model = dict(get_config("cfg2")["model"], block_kind=kind)
    nb = R.num_blocks(model)
    params = make_params(model, 0, perturb_bn=True)
    for b in (-1, 0, 1, 3, nb - 1, nb):
        lay = R.block_layout(model, b)
        assert sum(t["count"] for t in lay if t["kind"] not in (3, 4)) == OR.param_count(model, b)
        assert sum(t["count"] for t in lay) == OR.param_count(model, b, trainable_only=False)
        back = R.unpack_block(model, b, R.pack_block(model, b, params[b]))
        assert set(back) == set(params[b])
        for k in back:
            np.testing.assert_array_equal(back[k], params[b][k])
    # a BN of a pre-activation block has its convolution's INPUT channels
    first_of_stage2 = model["blocks"][0]
    lay = {(t["kind"], t["layer"]): t for t in R.block_layout(model, first_of_stage2)}
    assert lay[(1, 0)]["dims"][0] == lay[(0, 0)]["dims"][3]
    assert (1, 3) not in lay and (0, 3) in lay            # the shortcut convolution has no BN
    with pytest.raises(R.ResistError, match="stem"):
        R.num_blocks(dict(model, stem_kind=1))
    assert R.workspace_bytes(model, [0, 3, 7, 30], 8) > 0


def test_forward_and_aggregate_argument_errors():
    """Validation happens before any kernel is launched, so the error paths run without a GPU."""
    model = get_config("cfg2")["model"]
    d = R.model_desc(model)
    lib = R.lib()
    blocks = (ctypes.c_int32 * 4)(0, 3, 7, 30)
    n = ctypes.c_int64()
    assert lib.resist_forward_workspace_bytes(ctypes.byref(d), blocks, 4, 8, ctypes.byref(n)) == 0 and n.value > 0
    assert lib.resist_forward_workspace_bytes(ctypes.byref(d), blocks, 3, 8, ctypes.byref(n)) == -2      # stage 4's first block missing
    assert lib.resist_forward_workspace_bytes(ctypes.byref(d), blocks, 4, 8, None) == -1
    rc = lib.resist_forward(ctypes.byref(d), blocks, 4, None, None, None, 8, None, 0, None, None, None, None)
    assert rc == -1
    # labels without a loss buffer (fake, never dereferenced: the call fails before that)
    fake = (ctypes.c_void_p * 6)(*([16] * 6))
    rc = lib.resist_forward(ctypes.byref(d), blocks, 4, fake, None, ctypes.c_void_p(16), 8, ctypes.c_void_p(16), 1 << 40,
                            ctypes.c_void_p(16), ctypes.c_void_p(16), None, None)
    assert rc == -1 and b"labels" in lib.resist_last_error()
    # workspace too small
    rc = lib.resist_forward(ctypes.byref(d), blocks, 4, fake, None, ctypes.c_void_p(16), 8, ctypes.c_void_p(16), 1024,
                            ctypes.c_void_p(16), None, None, None)
    assert rc == -3
    # misaligned parameter buffer
    bad = (ctypes.c_void_p * 6)(16, 16, 20, 16, 16, 16)
    rc = lib.resist_forward(ctypes.byref(d), blocks, 4, bad, None, ctypes.c_void_p(16), 8, ctypes.c_void_p(16), 1 << 40,
                            ctypes.c_void_p(16), None, None, None)
    assert rc == -1
    # aggregate: S < 1, too many holders, block index out of range
    nb = R.num_blocks(model)
    offs = (ctypes.c_int32 * 2)(0, 4)
    glob = (ctypes.c_void_p * (nb + 2))(*([16] * (nb + 2)))
    one = (ctypes.POINTER(ctypes.c_void_p) * 1)(ctypes.cast(fake, ctypes.POINTER(ctypes.c_void_p)))
    assert lib.resist_aggregate(ctypes.byref(d), 0, offs, blocks, one, glob, None) == -1
    assert lib.resist_aggregate(ctypes.byref(d), 17, offs, blocks, one, glob, None) == -5
    badblocks = (ctypes.c_int32 * 4)(0, 3, 7, 99)
    assert lib.resist_aggregate(ctypes.byref(d), 1, offs, badblocks, one, glob, None) == -1
    # bf16 layer entry points refuse channel counts that are not multiples of 8
    from paper_2107_00961_amd.binding import _conv_shape
    sh = _conv_shape(1, 4, 4, 12, 16, 3, 1, 1, 1)
    rc = lib.resist_conv2d_forward(ctypes.byref(sh), ctypes.c_void_p(16), ctypes.c_void_p(16), ctypes.c_void_p(16), None, 0, None)
    assert rc == -2


def test_tensors_beyond_two_gib_are_refused_up_front():
    """The kernels address a tensor with 32-bit byte offsets: a batch that would push any activation
    past 2 GiB is refused when the plan is made (maximum sizes), in fp32 earlier than in bf16."""
    model = get_config("cfg2")["model"]                     # stem output: batch x 32 x 32 x 64 floats
    blocks = [0, 3, 7, 30]
    assert R.workspace_bytes(model, blocks, 8191) > 0      # 8191 * 65536 * 4 B just under 2 GiB
    with pytest.raises(R.ResistError, match="2 GiB"):
        R.workspace_bytes(model, blocks, 8192)
    bf = dict(model, compute_dtype=1)
    assert R.workspace_bytes(bf, blocks, 8192) > 0
    with pytest.raises(R.ResistError, match="2 GiB"):
        R.workspace_bytes(bf, blocks, 16384)
    with pytest.raises(R.ResistError, match="2 GiB"):
        R.forward_workspace_bytes(model, blocks, 8192)
    with pytest.raises(R.ResistError, match="2 GiB"):
        R.workspace_bytes(dict(model, block_kind=2), blocks, 8192)


def test_compressed_block_sizes_and_argument_errors():
    """Sizes of a compressed block follow the layout (one code per float of the buffer, a byte or a
    nibble each; one header record per tensor); bad arguments are refused before any launch."""
    lib = R.lib()
    for kind in (0, 1, 2, 3):
        model = dict(get_config("cfg2")["model"], block_kind=kind, num_classes=7)
        nb = R.num_blocks(model)
        for key in (-1, 0, 3, nb - 1, nb):
            n_total = R.block_param_count(model, key)[0]
            nt = len(R.block_layout(model, key))
            for bits in (8, 5):
                assert R.compressed_block_size(model, key, bits) == (n_total, nt)
            for bits in (4, 2):
                assert R.compressed_block_size(model, key, bits) == ((n_total + 1) // 2, nt)
    model = get_config("cfg2")["model"]
    d = R.model_desc(model)
    for bits in (1, 9, 0, -3):
        with pytest.raises(R.ResistError, match="bits"):
            R.compressed_block_size(model, 0, bits)
    with pytest.raises(R.ResistError):
        R.compressed_block_size(model, R.num_blocks(model) + 1, 8)
    keys = (ctypes.c_int32 * 2)(0, 1)
    ok = (ctypes.c_void_p * 2)(256, 256)
    assert lib.resist_compress_blocks(ctypes.byref(d), 2, keys, 8, None, ok, ok, None) == -1
    assert lib.resist_compress_blocks(ctypes.byref(d), 2, keys, 8, ok, (ctypes.c_void_p * 2)(256, 0), ok, None) == -1
    assert lib.resist_compress_blocks(ctypes.byref(d), 2, keys, 8, ok, (ctypes.c_void_p * 2)(256, 258), ok, None) == -1   # codes not 4-byte aligned
    assert lib.resist_compress_blocks(ctypes.byref(d), 2, keys, 8, ok, ok, (ctypes.c_void_p * 2)(256, 264), None) == -1   # header not 16-byte aligned
    assert lib.resist_compress_blocks(ctypes.byref(d), 2, keys, 12, ok, ok, ok, None) == -1
    assert lib.resist_compress_blocks(ctypes.byref(d), 0, None, 8, None, None, None, None) == 0                         # nothing to do
    assert lib.resist_decompress_blocks(ctypes.byref(d), 2, keys, 8, ok, ok, None, None) == -1
    assert lib.resist_decompress_blocks(ctypes.byref(d), 2, keys, 8, ok, ok, (ctypes.c_void_p * 2)(256, 260), None) == -1  # params not 16-byte aligned
    assert lib.resist_decompress_blocks(ctypes.byref(d), 2, keys, 1, ok, ok, ok, None) == -1
    assert lib.resist_decompress_blocks(ctypes.byref(d), 0, None, 8, None, None, None, None) == 0
    assert lib.resist_set_overlap(3) == -1 and lib.resist_set_overlap(1) == 0
    assert lib.resist_set_bn_fusion(3) == -1 and lib.resist_set_bn_fusion(-1) == -1 and lib.resist_set_bn_fusion(1) == 0
    nb = R.num_blocks(model)
    blocks = (ctypes.c_int32 * 4)(0, 3, 7, 30)
    offs = (ctypes.c_int32 * 2)(0, 4)
    glob = (ctypes.c_void_p * (nb + 2))(*([256] * (nb + 2)))
    six = (ctypes.c_void_p * 6)(*([256] * 6))
    one = (ctypes.POINTER(ctypes.c_void_p) * 1)(ctypes.cast(six, ctypes.POINTER(ctypes.c_void_p)))
    assert lib.resist_aggregate_compressed(ctypes.byref(d), 0, offs, blocks, 8, one, one, glob, None) == -1
    assert lib.resist_aggregate_compressed(ctypes.byref(d), 17, offs, blocks, 8, one, one, glob, None) == -5
    assert lib.resist_aggregate_compressed(ctypes.byref(d), 1, offs, blocks, 9, one, one, glob, None) == -1
    assert lib.resist_aggregate_compressed(ctypes.byref(d), 1, offs, blocks, 8, one, None, glob, None) == -1
    bad = (ctypes.c_int32 * 4)(0, 3, 3, 30)
    assert lib.resist_aggregate_compressed(ctypes.byref(d), 1, offs, bad, 8, one, one, glob, None) == -1                # not ascending
