#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<32>(const ColumnsCall &);
template int columns_plane_n1<36>(const ColumnsCall &);
template int columns_plane_n1<40>(const ColumnsCall &);
}  // namespace apw
