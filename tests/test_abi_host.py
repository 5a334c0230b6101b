"""Host side of the C ABI, no device needed: the library loads, exports every
symbol the header declares, and rejects bad requests with the documented
status codes before enqueueing anything (fake device addresses are never
dereferenced on these paths)."""
import ctypes as C
import os
import re

import pytest

from paper_2608_10139_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000   # never dereferenced: plan creation only records addresses


def header_functions():
    src = open(os.path.join(ROOT, "include", "aiq.h")).read()
    return sorted(set(re.findall(r"\b(aiq_[a-z_]+)\s*\(", src)) - {"aiq_status"})


def test_library_exports_every_declared_function():
    lib = B.load()
    declared = header_functions()
    assert set(declared) == set(B.EXPORTS)
    for fn in declared:
        assert hasattr(lib, fn), fn
    header = open(os.path.join(ROOT, "include", "aiq.h")).read()
    declared_version = int(re.search(r"#define AIQ_ABI_VERSION (\d+)", header).group(1))
    assert B.aiq_abi_version() == declared_version == B.AIQ_ABI_VERSION
    assert B.aiq_status_str(B.AIQ_ENOSPC) == "workspace or capacity too small"


def model(**kw):
    m = B.aiq_model()
    m.n_layers, m.d_model, m.n_heads, m.n_kv_heads, m.d_ff, m.vocab = 2, 512, 8, 8, 2048, 32000
    m.act, m.wdtype, m.rope_theta, m.norm_eps = B.AIQ_ACT_SWIGLU, B.AIQ_BF16, 10000.0, 1e-5
    m.emb = m.final_norm = m.lm_head = FAKE
    layers = (B.aiq_layer * 2)()
    for L in layers:
        for f, _ in B.aiq_layer._fields_:
            setattr(L, f, FAKE)
    m.layers = C.cast(layers, C.POINTER(B.aiq_layer))
    m._keep = layers
    for k, v in kw.items():
        setattr(m, k, v)
    return m


def table(n=1000):
    cols = (B.aiq_col * 2)()
    cols[0].data, cols[0].dtype = FAKE, B.AIQ_I8
    cols[1].data, cols[1].dtype = FAKE, B.AIQ_I32
    t = B.aiq_table()
    t.n_rows, t.n_cols, t.cols = n, 2, C.cast(cols, C.POINTER(B.aiq_col))
    t.list_offsets = t.list_tokens = FAKE
    t.n_list_tokens, t.max_list_len = n * 100, 512
    t._keep = cols
    return t


def query(**kw):
    q = B.aiq_query()
    q.n_pred = 1
    q.preds[0].col, q.preds[0].op, q.preds[0].k = 0, B.AIQ_LE, 2
    q.n_labels, q.label_ids[0], q.label_ids[1] = 2, 1, 2
    q.decision, q.agg = B.AIQ_DECIDE_BINARY_GT, B.AIQ_AGG_COUNT
    for k, v in kw.items():
        setattr(q, k, v)
    return q


def test_16_bit_models_reserve_no_rotary_tables():
    """Their projections take the angles from the frequencies of a head's dims; the
    cos / sin tables (8 bytes per position and pair of dims) belong to the fp32
    path.  Heads of 64 and of 128 with the same widths need the same workspace
    (but for the frequencies, one 256-byte block either way)."""
    plans = [B.aiq_plan_create(model(n_heads=h, n_kv_heads=h), table(), None, query()) for h in (8, 4)]
    try:
        for size in (B.aiq_workspace_size, lambda p: B.aiq_prefill_workspace_size(p, 4096)):
            assert size(plans[0]) == size(plans[1])
    finally:
        for p in plans:
            B.aiq_plan_destroy(p)


def test_valid_plan_and_workspace_size():
    p = B.aiq_plan_create(model(), table(), None, query())
    try:
        n = B.aiq_workspace_size(p)
        assert n > 0
        assert B.aiq_prefill_workspace_size(p, 4096) > 0
    finally:
        B.aiq_plan_destroy(p)


@pytest.mark.parametrize("field,value,code", [
    ("d_model", 500, B.AIQ_EINVAL),          # d % n_heads
    ("n_kv_heads", 3, B.AIQ_EINVAL),         # n_heads % n_kv
    ("d_model", 8 * 48, B.AIQ_EINVAL),       # head dim 48
    ("wdtype", 9, B.AIQ_EINVAL),
    ("act", 7, B.AIQ_EINVAL),
    ("emb", 0, B.AIQ_EINVAL),
    ("norm_eps", 0.0, B.AIQ_EINVAL),
    ("act", B.AIQ_ACT_GELU_ERF, B.AIQ_EUNSUPPORTED),   # bf16 path is SwiGLU only
])
def test_model_validation(field, value, code):
    assert B.aiq_plan_create_status(model(**{field: value}), table(), None, query()) == code


def test_null_model_and_bad_query():
    assert B.aiq_plan_create_status(None, table(), None, query()) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, query(n_labels=1)) == B.AIQ_EINVAL
    q = query(); q.preds[0].col = 5
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_EINVAL
    q = query(); q.preds[0].op = 42
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_EINVAL
    q = query(); q.label_ids[1] = 32000
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_EINVAL
    # a join without a build table, and a build table without a join
    assert B.aiq_plan_create_status(model(), table(), None, query(join=1)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), table(), query()) == B.AIQ_EINVAL
    # group-by: a dense key domain (n_group_keys > 0) or any int32 key (0); not negative
    assert B.aiq_plan_create_status(model(), table(), None, query(agg=B.AIQ_AGG_AVG_LABEL_COUNT_BY,
                                                                  group_col=1, n_group_keys=-1)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, query(agg=B.AIQ_AGG_AVG_LABEL_COUNT_BY,
                                                                  group_col=1)) == B.AIQ_OK
    # count-by-payload needs a join
    assert B.aiq_plan_create_status(model(), table(), None, query(agg=B.AIQ_AGG_COUNT_BY_PAYLOAD,
                                                                  n_group_keys=4)) == B.AIQ_EINVAL


def test_table_validation():
    t = table(); t.cols[1].data = FAKE + 4   # columns must be 16-byte aligned
    assert B.aiq_plan_create_status(model(), t, None, query()) == B.AIQ_EINVAL
    t = table(); t.list_offsets = 0
    assert B.aiq_plan_create_status(model(), t, None, query()) == B.AIQ_EINVAL
    t = table(); t.max_list_len = 0
    assert B.aiq_plan_create_status(model(), t, None, query()) == B.AIQ_EINVAL
    t = table(); t.n_rows = -1
    assert B.aiq_plan_create_status(model(), t, None, query()) == B.AIQ_EINVAL


def float_table(n=1000):
    t = table(n)
    t.cols[1].dtype = B.AIQ_F32
    return t


def test_float_column_rules():
    q = query()
    q.preds[0].col, q.preds[0].op, q.preds[0].fk = 1, B.AIQ_GT, 70.0
    assert B.aiq_plan_create_status(model(), float_table(), None, q) == B.AIQ_OK
    q.preds[0].op, q.preds[0].n_set = B.AIQ_IN, 1          # IN is integer-only
    assert B.aiq_plan_create_status(model(), float_table(), None, q) == B.AIQ_EUNSUPPORTED
    # SUM needs an fp32 column
    assert B.aiq_plan_create_status(model(), float_table(), None,
                                    query(agg=B.AIQ_AGG_SUM_F32, group_col=1)) == B.AIQ_OK
    assert B.aiq_plan_create_status(model(), float_table(), None,
                                    query(agg=B.AIQ_AGG_SUM_F32, group_col=0)) == B.AIQ_EUNSUPPORTED
    # a relational-only plan has no labels to sum over
    o = _opts(B.AIQ_PLAN_RELATIONAL_ONLY)
    assert B.aiq_plan_create_status(model(), float_table(), None,
                                    query(agg=B.AIQ_AGG_SUM_F32, group_col=1), o) == B.AIQ_EINVAL


def test_sum_run_needs_output():
    lib = B.load()
    p = B.aiq_plan_create(model(), float_table(), None, query(agg=B.AIQ_AGG_SUM_F32, group_col=1))
    try:
        need = B.aiq_workspace_size(p)
        out = B.aiq_out()
        out.scalars, out.ids, out.ids_cap = FAKE, FAKE, 1000
        assert lib.aiq_run(p, FAKE, need, C.byref(out), None, None) == B.AIQ_EINVAL   # no sum_out
    finally:
        B.aiq_plan_destroy(p)


def _opts(flags):
    o = B.aiq_plan_opts()
    o.flags = flags
    return o


def test_relational_only_plan_validation():
    # the token column is optional only when the plan stops after the relational part
    t = table(); t.list_tokens = 0
    assert B.aiq_plan_create_status(model(), t, None, query()) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), t, None, query(), _opts(B.AIQ_PLAN_RELATIONAL_ONLY)) == B.AIQ_OK
    # offsets stay required (token counts come from them)
    t = table(); t.list_offsets = 0
    assert B.aiq_plan_create_status(model(), t, None, query(), _opts(B.AIQ_PLAN_RELATIONAL_ONLY)) == B.AIQ_EINVAL
    # only COUNT: there are no labels to aggregate
    q = query(agg=B.AIQ_AGG_AVG_LABEL_COUNT_BY, group_col=1, n_group_keys=4)
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_OK
    assert B.aiq_plan_create_status(model(), table(), None, q, _opts(B.AIQ_PLAN_RELATIONAL_ONLY)) == B.AIQ_EINVAL
    # unknown flag bits
    assert B.aiq_plan_create_status(model(), table(), None, query(), _opts(16)) == B.AIQ_EINVAL
    for flag in (B.AIQ_PLAN_MULTIPASS_COMPACT, B.AIQ_PLAN_FULL_LAST_LAYER):
        assert B.aiq_plan_create_status(model(), table(), None, query(), _opts(flag)) == B.AIQ_OK
    assert B.aiq_plan_create_status(model(), table(), None, query(), _opts(B.AIQ_PLAN_UNSHARED_PREFIX)) == B.AIQ_OK


def _prefix_query(n):
    q = query()
    q.n_prefix = n
    for k in range(n):
        q.prefix[k] = 3 + k
    return q


def test_plan_passes():
    shared = B.aiq_plan_create(model(), table(), None, _prefix_query(32))
    unshared = B.aiq_plan_create(model(), table(), None, _prefix_query(32), _opts(B.AIQ_PLAN_UNSHARED_PREFIX))
    rel = B.aiq_plan_create(model(), table(), None, query(), _opts(B.AIQ_PLAN_RELATIONAL_ONLY))
    small = B.aiq_plan_opts()
    small.chunk_tokens = 10_000
    chunked = B.aiq_plan_create(model(), table(), None, query(), small)
    try:
        assert B.aiq_plan_passes(shared) == (1, 1)
        assert B.aiq_plan_passes(unshared) == (1, 0)
        assert B.aiq_plan_passes(rel) == (0, 0)
        # 100,000 table tokens plus one unit per row (1,000 rows) in chunks of 10,000
        assert B.aiq_plan_passes(chunked) == (11, 0)
    finally:
        for p in (shared, unshared, rel, chunked):
            B.aiq_plan_destroy(p)


def test_last_layer_rows_plan_flag():
    """16-bit models run the last layer for the last positions only unless
    AIQ_PLAN_FULL_LAST_LAYER; fp32 models and zero-layer plans never do."""
    plans = {
        "default": B.aiq_plan_create(model(), table(), None, query()),
        "full": B.aiq_plan_create(model(), table(), None, query(), _opts(B.AIQ_PLAN_FULL_LAST_LAYER)),
        "fp32": B.aiq_plan_create(model(wdtype=B.AIQ_F32, act=B.AIQ_ACT_GELU_ERF), table(), None, query()),
    }
    no_layer = B.aiq_plan_opts()
    no_layer.n_layers_override = -1
    plans["no_layer"] = B.aiq_plan_create(model(), table(), None, query(), no_layer)
    try:
        assert B.aiq_plan_last_layer_rows(plans["default"]) is True
        assert B.aiq_plan_last_layer_rows(plans["full"]) is False
        assert B.aiq_plan_last_layer_rows(plans["fp32"]) is False
        assert B.aiq_plan_last_layer_rows(plans["no_layer"]) is False
        # the pruned plan needs the compact last-layer rows on top
        assert B.aiq_workspace_size(plans["default"]) > B.aiq_workspace_size(plans["full"])
    finally:
        for p in plans.values():
            B.aiq_plan_destroy(p)


def test_shared_prefix_is_packed_once():
    # 1000 rows of 100 tokens with a 32-token prompt: the shared plan packs
    # the 100,000 row tokens only (plus per-layer prefix keys / values), the
    # unshared plan 132,000 tokens, and every per-token buffer grows with that
    shared = B.aiq_plan_create(model(), table(), None, _prefix_query(32))
    unshared = B.aiq_plan_create(model(), table(), None, _prefix_query(32), _opts(B.AIQ_PLAN_UNSHARED_PREFIX))
    plain = B.aiq_plan_create(model(), table(), None, query())
    try:
        ws, wu, wp = (B.aiq_workspace_size(p) for p in (shared, unshared, plain))
        assert wp <= ws < wu
        # the shared plan adds only the prefix's per-layer q|k|v rows and its small batch
        d, n_qkv, layers = 512, 512 * 3, 2
        assert ws - wp <= layers * 32 * n_qkv * 2 + 32 * 4 + d * 4 + 4 * 4096
    finally:
        for p in (shared, unshared, plain):
            B.aiq_plan_destroy(p)


def test_relational_only_workspace_holds_no_model_activations():
    full = B.aiq_plan_create(model(), table(), None, query())
    rel = B.aiq_plan_create(model(), table(), None, query(), _opts(B.AIQ_PLAN_RELATIONAL_ONLY))
    try:
        # 1000 rows x 100 tokens: the full plan carries the packed batch and the activations
        assert B.aiq_workspace_size(rel) < B.aiq_workspace_size(full) // 10
    finally:
        B.aiq_plan_destroy(full)
        B.aiq_plan_destroy(rel)


def test_run_rejects_before_enqueue():
    p = B.aiq_plan_create(model(), table(), None, query())
    try:
        need = B.aiq_workspace_size(p)
        out = B.aiq_out()
        out.scalars, out.ids, out.ids_cap = FAKE, FAKE, 1000
        lib = B.load()
        assert lib.aiq_run(p, FAKE, need - 1, C.byref(out), None, None) == B.AIQ_ENOSPC
        assert lib.aiq_run(p, None, need, C.byref(out), None, None) == B.AIQ_EINVAL
        assert lib.aiq_run(None, FAKE, need, C.byref(out), None, None) == B.AIQ_EINVAL
        out.scalars = 0
        assert lib.aiq_run(p, FAKE, need, C.byref(out), None, None) == B.AIQ_EINVAL
        assert lib.aiq_prefill_packed(p, FAKE, FAKE, 0, 10, B.AIQ_LOGITS_LABELS, FAKE, FAKE, 1 << 30, None) == B.AIQ_EINVAL
        assert lib.aiq_prefill_packed(p, FAKE, FAKE, 2, 10, 9, FAKE, FAKE, 1 << 30, None) == B.AIQ_EINVAL
        assert lib.aiq_prefill_packed(p, FAKE, FAKE, 2, 10, B.AIQ_LOGITS_LABELS, FAKE, FAKE, 16, None) == B.AIQ_ENOSPC
    finally:
        B.aiq_plan_destroy(p)


def _gen_query(**kw):
    q = query(n_labels=0, gen_tokens=16, eos_id=2, pad_id=0)
    for k, v in kw.items():
        setattr(q, k, v)
    return q


def test_transform_plan_validation():
    ok = B.AIQ_OK
    # labels are not needed for generation
    assert B.aiq_plan_create_status(model(), table(), None, _gen_query()) == ok
    assert B.aiq_plan_create_status(model(), table(), None, _gen_query(gen_tokens=B.AIQ_MAX_GEN + 1)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _gen_query(gen_tokens=-1)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _gen_query(eos_id=32000)) == B.AIQ_EINVAL
    q = _gen_query(n_like=2)
    q.like[0], q.like[1] = 5, 32000
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_EINVAL
    q.like[1] = 6
    assert B.aiq_plan_create_status(model(), table(), None, q) == ok
    assert B.aiq_plan_create_status(model(), table(), None, _gen_query(n_like=B.AIQ_MAX_LIKE + 1)) == B.AIQ_EINVAL
    # fp32 models and vocabularies that the full-vocabulary head cannot tile
    assert B.aiq_plan_create_status(model(wdtype=B.AIQ_F32), table(), None, _gen_query()) == B.AIQ_EUNSUPPORTED
    assert B.aiq_plan_create_status(model(vocab=32001), table(), None, _gen_query()) == B.AIQ_EUNSUPPORTED
    # no label to average
    q = _gen_query(agg=B.AIQ_AGG_AVG_LABEL_COUNT_BY, group_col=1, n_group_keys=4)
    assert B.aiq_plan_create_status(model(), table(), None, q) == B.AIQ_EINVAL


def test_transform_workspace_holds_the_generation_state():
    plain = B.aiq_plan_create(model(), table(), None, query())
    g16 = B.aiq_plan_create(model(), table(), None, _gen_query(gen_tokens=16))
    g32 = B.aiq_plan_create(model(), table(), None, _gen_query(gen_tokens=32))
    try:
        wp, w16, w32 = (B.aiq_workspace_size(p) for p in (plain, g16, g32))
        assert wp < w16 < w32
        # 16 more slots per row in the generated-token cache: 2 layers x 1000
        # rows x 16 x 2 * 512 fp16 values, and 16 more token ids per row
        assert w32 - w16 >= 2 * 1000 * 16 * 2 * 512 * 2 + 1000 * 16 * 4
    finally:
        for p in (plain, g16, g32):
            B.aiq_plan_destroy(p)


def _pair_query(**kw):
    q = query(pairs=1, pair_key_col=1, n_group_keys=100, max_pairs=5000)
    for k, v in kw.items():
        setattr(q, k, v)
    return q


def test_pairs_plan_validation():
    ok = B.AIQ_OK
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query()) == ok
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(pairs=2)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(pair_key_col=2)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(max_pairs=0)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(n_group_keys=0)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(n_group_keys=16385)) == B.AIQ_EUNSUPPORTED
    assert B.aiq_plan_create_status(model(), table(), None,
                                    _pair_query(decision=B.AIQ_DECIDE_ARGMAX)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(gen_tokens=4)) == B.AIQ_EINVAL
    assert B.aiq_plan_create_status(model(), table(), None, _pair_query(),
                                    _opts(B.AIQ_PLAN_RELATIONAL_ONLY)) == B.AIQ_EINVAL


def test_pairs_workspace_follows_max_pairs():
    small = B.aiq_plan_create(model(), table(), None, _pair_query(max_pairs=1000))
    big = B.aiq_plan_create(model(), table(), None, _pair_query(max_pairs=2000))
    try:
        # 1000 more pairs of up to 2 x 512 tokens each, packed as int32
        assert B.aiq_workspace_size(big) - B.aiq_workspace_size(small) >= 1000 * 1024 * 4
    finally:
        B.aiq_plan_destroy(small)
        B.aiq_plan_destroy(big)


def test_relational_static_refusals():
    """The entry point without a workspace refuses, before enqueuing
    anything: a plan that is not relational-only, and a plan whose scratch
    (here a 2^21-row build table: 2^22 hash slots, 32 MiB) exceeds the fixed
    16 MiB array."""
    out = B.aiq_out()
    sc = (C.c_int64 * B.AIQ_N_SCALARS)()
    out.scalars = C.cast(sc, C.c_void_p)
    full = B.aiq_plan_create(model(), table(), None, query())
    try:
        assert B.aiq_run_relational_static_status(full, out) == B.AIQ_EINVAL
    finally:
        B.aiq_plan_destroy(full)
    bcols = (B.aiq_col * 2)()
    bcols[0].data, bcols[0].dtype = FAKE, B.AIQ_I32
    bcols[1].data, bcols[1].dtype = FAKE, B.AIQ_I8
    build = B.aiq_table()
    build.n_rows, build.n_cols, build.cols = 1 << 21, 2, C.cast(bcols, C.POINTER(B.aiq_col))
    q = query()
    q.join, q.probe_key_col, q.build_key_col, q.build_payload_col = 1, 1, 0, 1
    big = B.aiq_plan_create(model(), table(), build, q, _opts(B.AIQ_PLAN_RELATIONAL_ONLY))
    try:
        assert B.aiq_run_relational_static_status(big, out) == B.AIQ_ENOSPC
    finally:
        B.aiq_plan_destroy(big)


def test_convert_weights_refusals():
    """Refused before anything is enqueued: another pair of types, a negative
    count, a NULL pointer with elements, a misaligned pointer."""
    assert B.load().aiq_convert_weights(FAKE, B.AIQ_F16, FAKE, B.AIQ_BF16, 8, None) == B.AIQ_EUNSUPPORTED
    assert B.load().aiq_convert_weights(FAKE, B.AIQ_BF16, FAKE, B.AIQ_F16, -1, None) == B.AIQ_EINVAL
    assert B.load().aiq_convert_weights(None, B.AIQ_BF16, FAKE, B.AIQ_F16, 8, None) == B.AIQ_EINVAL
    assert B.load().aiq_convert_weights(FAKE + 2, B.AIQ_BF16, FAKE, B.AIQ_F16, 8, None) == B.AIQ_EINVAL
