// The layout that the library gives a descriptor, for tests (CPU only): its host code with nothing else
// of the library, compiled where a test asks for it.
#include "../paper_2609_32922_amd/csrc/sc_api.hip"

// what: 0 sc_gemm's layout, 1 the tables of a C-BSG call behind its planes.  Returns SC_OK, an error, or 1
// where there are no tables.
extern "C" __attribute__((visibility("default"))) int layout_query(const sc_gemm_desc *d, int cus, int what, int64_t *o) {
    const int rc = check_desc(d);
    if (rc != SC_OK) return rc;
    Layout l, t;
    if (!make_layout(*d, cus, &l)) return SC_ERR_SHAPE;
    if (what == 1) {
        if (!make_cbsg_layout(*d, cus, l, &t)) return 1;
        l = t;
    }
    const int64_t v[] = {(int64_t)l.total, l.rgen, l.tall, l.narrow, l.fused, l.S, l.F, l.p16, l.vsplit, l.sk_slots, l.nplans};
    for (size_t k = 0; k < sizeof(v) / sizeof(v[0]); ++k) o[k] = v[k];
    return SC_OK;
}
