"""GPU parity at the benchmarked sizes, in the launch configurations the
benchmark times.

Each test encodes a whole benchmarked micro-batch (the same seeded request
pools as bench.py) and checks sampled requests against the fp64 reference run
on that request alone, at full depth where the reference finishes in seconds
and at two layers otherwise; it also checks that each sampled request's rows
are bit-identical to its own micro-batch-1 encoding.  From 8192 tokens a
micro-batch runs as two concurrent halves on two streams, the GEMMs run the
large-tile path, including the split of quantised grids into a 256 x 256 head
launch and a smaller-tile tail launch, and attention runs over the longest
sequences (9216-token images, 8192-token clips); CLIP x8 runs in one pass on
smaller tiles.
"""
import numpy as np
import pytest

from _harness import TOL, gpu_encode, oracle_encode, rel_err
from paper_2609_31551_amd import configs as C
from paper_2609_31551_amd import synth

pytestmark = pytest.mark.gpu


def _check_samples(p, items, W, samples, max_tokens=None):
    batch = gpu_encode(p, items, W, max_tokens=max_tokens)
    cu = batch["cu_out"]
    for r in samples:
        print("[full-size] %s: request %d of %d" % (p["name"], r, len(items)), flush=True)
        ref = oracle_encode(p, [items[r]], W)
        e = rel_err(batch["out"][cu[r]:cu[r + 1]], ref["out"])
        print("[full-size] %s: request %d relative error %.3g" % (p["name"], r, e), flush=True)
        assert e <= TOL[p["dtype"]], (r, e)
        alone = gpu_encode(p, [items[r]], W, enc=batch["enc"], wdev=batch["wdev"])
        np.testing.assert_array_equal(alone["out"], batch["out"][cu[r]:cu[r + 1]])


def test_clip_microbatch_64_full_depth():
    """The headline workload: 64 CLIP images (36928 tokens), full depth;
    request 63 sits in the rows of the tail launches of the split GEMMs."""
    p = C.CLIP_L336
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 64, 0)
    _check_samples(p, items, W, [5, 63])


def test_clip_microbatch_8_full_depth():
    """The first 8 images of the CLIP pool (4616 tokens, one pass: the
    O-projection on 128 x 128 persistent tiles, FC2 on 192 x 128 deep ones), full depth."""
    p = C.CLIP_L336
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 64, 0)[:8]
    _check_samples(p, items, W, [0, 7])


def test_clip_microbatch_32_full_depth():
    """The first 32 images of the CLIP pool (18464 tokens: two halves of 16
    images), full depth."""
    p = C.CLIP_L336
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 64, 0)[:32]
    _check_samples(p, items, W, [15, 31])


def test_single_requests_full_depth():
    """Micro-batch 1 (the low-load end of the sweep), full depth: one CLIP image
    (577 tokens) and one audio clip (1500 tokens).  Every GEMM of their layers but
    the clip's FC1 then runs the deep-pipelined kernel, on its four tiles between
    them; the batched encodings of the same requests (CLIP x8, audio x8) must match them
    bit for bit."""
    for p, pool, r in ((C.CLIP_L336, 64, 3), (C.WHISPER_L, 32, 2)):
        W = synth.make_weights(p, 0)
        items = synth.make_items(p, pool, 0)[:8]
        print("[full-size] %s: request %d alone" % (p["name"], r), flush=True)
        alone = gpu_encode(p, [items[r]], W)
        ref = oracle_encode(p, [items[r]], W)
        e = rel_err(alone["out"], ref["out"])
        print("[full-size] %s: request %d alone, relative error %.3g" % (p["name"], r, e), flush=True)
        assert e <= TOL[p["dtype"]], (p["name"], e)
        batch = gpu_encode(p, items, W)
        cu = batch["cu_out"]
        np.testing.assert_array_equal(alone["out"], batch["out"][cu[r]:cu[r + 1]])


def test_whisper_microbatch_8_full_depth():
    """The first 8 clips of the audio pool (12000 tokens: two halves), full depth."""
    p = C.WHISPER_L
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 32, 0)[:8]
    _check_samples(p, items, W, [7])


def test_qwen_image_microbatch_8_full_depth():
    """The first 8 images of the 64-image pool (variable resolution), full
    depth; the smallest image is checked against the reference."""
    p = C.QWEN_IMAGE
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 64, 0)[:8]
    sizes = [a.shape[2] * a.shape[3] for a in items]
    _check_samples(p, items, W, [int(np.argmin(sizes))])


def test_qwen_image_microbatch_32_full_depth():
    """The largest swept micro-batch of the image workload: the first 32 images
    of the 64-image pool, full depth; the smallest image is checked against the
    reference."""
    p = C.QWEN_IMAGE
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 64, 0)[:32]
    sizes = [a.shape[2] * a.shape[3] for a in items]
    _check_samples(p, items, W, [int(np.argmin(sizes))])


def test_qwen_image_largest_images_two_layers():
    """Micro-batch with 1344 x 1344 images (9216 tokens each, the longest
    attention rows of the image workload) at two layers."""
    p = C.with_layers(C.QWEN_IMAGE, 2)
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 3, 0, shapes=[(2, 1344, 1344), (2, 672, 1344), (2, 1344, 1344)])
    _check_samples(p, items, W, [2])


def test_largest_accepted_microbatch_two_layers():
    """The largest micro-batch a Qwen-style handle accepts (the 32-bit offset
    cap, 419430 tokens): 45 images of 1344 x 1344 (9216 tokens each) and a
    224 x 224 one (256 tokens) last, two layers, run as one pass (profiling
    on, so no split into halves): every launch spans whole buffers, and the
    last rows of the widest one (FC1's, 5120 columns) end about 1% below 2^31
    elements.  The small image, at the highest offsets, is checked against the
    reference and its own single encoding; the last large image against its
    single encoding."""
    from paper_2609_31551_amd import eas
    p = C.with_layers(C.QWEN_IMAGE, 2)
    W = synth.make_weights(p, 0)
    shapes = [(2, 1344, 1344)] * 45 + [(2, 224, 224)]
    items = synth.make_items(p, len(shapes), 0, shapes=shapes)
    enc = eas.Encoder(p, 419430, max_seqs=len(items))
    wdev = eas.upload_weights(enc.cfg, W)
    enc.profile_enable(True)
    batch = gpu_encode(p, items, W, enc=enc, wdev=wdev)
    enc.profile_enable(False)
    enc.profile_read()
    cu = batch["cu_out"]
    assert batch["cu"][-1] == 45 * 9216 + 256
    print("[full-size] largest micro-batch: %d tokens in one pass" % batch["cu"][-1], flush=True)
    ref = oracle_encode(p, [items[45]], W)
    e = rel_err(batch["out"][cu[45]:cu[46]], ref["out"])
    print("[full-size] largest micro-batch: last request relative error %.3g" % e, flush=True)
    assert e <= TOL[p["dtype"]], e
    for r in (44, 45):
        alone = gpu_encode(p, [items[r]], W, enc=enc, wdev=wdev)
        np.testing.assert_array_equal(alone["out"], batch["out"][cu[r]:cu[r + 1]])


def test_video_microbatch_4_two_layers():
    """4 clips of 16 x 448 x 448 (32768 tokens, 8192 per clip), two layers."""
    p = C.with_layers(C.QWEN_VIDEO, 2)
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 4, 0)
    _check_samples(p, items, W, [3])


def test_whisper_microbatch_32_full_depth():
    """32 audio clips (48000 tokens), full depth."""
    p = C.WHISPER_L
    W = synth.make_weights(p, 0)
    items = synth.make_items(p, 32, 0)
    _check_samples(p, items, W, [31])
