"""Calls whose stores are written through: the smallest that get each launch, and which kernel (its template arguments) that is.
tests/test_host_launches.py holds the table against what the library launches, tests/test_gpu_written_through.py runs it."""
NONE, ALL, BUT_COMBINED, BY_RECORD, FORWARDED = range(5)   # the library's Through


def few(threads, unroll, stores, parts):
    return f"chunk_few_kernelILi{threads}ELi{unroll}E{{op}}LNS_7ThroughE{stores}ELb{int(parts)}ELb0EE"


def group(unroll, stores):
    return f"chunk_group_kernelILi256ELi{unroll}E{{op}}Lb0ELNS_7ThroughE{stores}EE"


def flat(tile, unroll, stores):
    return f"chunk_flat_kernelILi1024ELi{tile}ELi{unroll}E{{op}}LNS_7ThroughE{stores}EE"


def ordered(stores):
    return f"chunk_ordered_kernelI{{op}}LNS_7ThroughE{stores}EE"


# records, chunk bytes, whether the call states them, name, kernel of SUM, kernel of COPY
APPLY = [(57, 65536, True, "parts", few(256, 2, ALL, True), few(256, 2, ALL, True)),
         (200, 66000, True, "parts off lines", few(256, 2, ALL, True), few(256, 2, ALL, True)),
         (100, 65536, False, "parts by record, small", few(256, 2, BY_RECORD, True), few(256, 2, BY_RECORD, True)),
         (100, 400000, False, "parts by record, large", few(256, 2, BY_RECORD, True), few(256, 2, BY_RECORD, True)),
         (200, 32768, True, "a workgroup a record", few(1024, 4, ALL, False), few(1024, 4, ALL, False)),
         (200, 16384, True, "a workgroup a small record", few(1024, 1, ALL, False), few(1024, 1, ALL, False)),
         (700, 4096, True, "group of one vector", group(1, ALL), group(1, ALL)),
         (700, 6000, True, "group of two off lines", group(2, ALL), group(2, ALL)),
         (400, 8192, True, "group of two", group(2, ALL), group(2, ALL)),
         (300, 65536, True, "group of four", group(4, ALL), group(4, ALL)),
         (3200, 4096, True, "tiles of eight", flat(8, 2, BUT_COMBINED), flat(8, 2, BUT_COMBINED)),
         (3200, 8192, True, "tiles of four", flat(4, 2, BUT_COMBINED), flat(4, 2, BUT_COMBINED)),
         (8192, 12288, True, "tiles of two", flat(2, 2, BUT_COMBINED), flat(2, 2, BUT_COMBINED)),
         (8200, 12288, True, "large tiles of two", None, flat(2, 2, FORWARDED)),
         (2100, 40960, True, "one record a tile", flat(1, 1, BUT_COMBINED), flat(1, 2, NONE)),
         (800, 131072, True, "ordered", ordered(ALL), ordered(ALL))]
# records, chunk bytes, name, kernel of SUM
FOLD = [(400, 4096, "group", "gather_group_kernelI{op}Lb0EE"),
        (3100, 4096, "tiles of eight", "chunk_gather_kernelILi1024ELi8ELi2E{op}LNS_5StoreE17EE"),
        (8400, 9008, "large tiles off lines", "chunk_gather_kernelILi1024ELi4ELi2E{op}LNS_5StoreE0EE"),
        (600, 65536, "one record a tile", "chunk_gather_kernelILi1024ELi1ELi2E{op}LNS_5StoreE17EE"),
        (800, 131072, "ordered", "gather_ordered_kernelI{op}E")]
