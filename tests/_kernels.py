"""The drafter's kernels by test hook.  By size alone small shapes reach one of them only: the lists of the drafter's tests name the
kernel that a row is for, and run it by the library's own rule and on the kernels of few rows or many as well."""
STREAM = {"DD_TUNE_BLOCK_STREAM": "1"}                # at most 64 query rows per kv head: the streaming kernel
MFMA = {"DD_TUNE_BLOCK_STREAM": "0"}                  # ... the MFMA kernel
WIDE = {"DD_TUNE_BLOCK_WIDE": "1"}                    # more than 64 rows: the wide kernel, on the row tiles of its own rule
WIDE128, WIDE256 = {"DD_TUNE_BLOCK_WIDE_ROWS": "128"}, {"DD_TUNE_BLOCK_WIDE_ROWS": "256"}
OFF_WIDE = {"DD_TUNE_BLOCK_WIDE": "0"}                # ... the MFMA kernel
SOLO = {"DD_TUNE_SOLO": "1"}                          # waves that stream keys of their own
DUO2, DUO4 = {"DD_TUNE_DUO": "2"}, {"DD_TUNE_DUO": "4"}      # two waves per SIMD, 64 / 128 rows per workgroup

# that kernel's forms (row blocks, parts of the head dims, waves as digits) by storage: (q and k, v, head dims) as dtype tags, 1 bf16, 2 e4m3
SOLO_FORMS = {(1, 1, 128): (114, 124, 128, 144, 148, 224), (2, 1, 128): (114, 124, 128, 144, 148, 228),
              (2, 2, 128): (114, 124, 128, 144, 148, 224, 228), (1, 1, 64): (114, 118, 124, 128)}


def solo_form(form, splits=1):
    return {"DD_TUNE_SOLO": "1", "DD_TUNE_SOLO_FORM": str(form), "DD_TUNE_BLOCK_SPLITS": str(splits)}


def with_splits(env, n):
    return dict(env, DD_TUNE_BLOCK_SPLITS=str(n))


def by_rule_and_elsewhere(rows, served):
    """`rows` ((..., env) each), then every row that has a kernel of its own by the library's rule, and those `served` accepts on the
    kernels of few rows and of many."""
    more = [r[:-1] + ({},) for r in rows if r[-1]]
    shapes = [r for i, r in enumerate(rows) if served(r) and r[:-1] not in [q[:-1] for q in rows[:i]]]
    more += [r[:-1] + (env,) for r in shapes for env in (SOLO, DUO2, DUO4)]
    return rows + [r for i, r in enumerate(more) if r not in rows and r not in more[:i]]
